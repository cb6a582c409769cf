"""GPU: the second half of the fused log-softmax, on rows of whole 16-byte pieces and of others, at the edges of the stretches that
a row is divided into, against the logits of the product in binary64."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [1, 3, 4, 255, 1024, 2000, 4095, 4096, 4097, 4100, 8188, 8192, 8193, 8196, 9999, 10000, 12289, 42000])
@pytest.mark.parametrize("B", [1, 2, 20, 64])
def test_rows_of_any_length(V, B):
    import torch

    import paper_1802_00150_amd as amq
    print("log-softmax rows V=%d B=%d" % (V, B), flush=True)
    H = 300
    g = torch.Generator(device="cuda:0").manual_seed(V + B)
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda:0")  # noqa: E731
    W = amq.quantize_weights(randn(V, H) * 0.2, 2, 2)
    bias, h = randn(V), torch.tanh(randn(B, H))
    logits = amq.binary_gemm(*W, H, *amq.quantize_activations(h, 2, 2), bias=bias)
    want = torch.log_softmax(logits.double(), dim=1)
    got = amq.softmax_layer(*W, H, bias, h, 2, 2)
    # logits and the log of their sum are rounded to binary32 each, and the logits of the two calls may differ in the last digits
    bound = 8 * 2.0 ** -24 * (logits.abs().max().item() + want.abs().max().item() + 1) * 2
    assert (got.double() - want).abs().max().item() <= bound
    apart = torch.full((B * V + 1,), float("nan"), device=h.device)  # rows that do not start at 16 bytes
    amq.softmax_layer(*W, H, bias, h, 2, 2, logprob=apart[1:].view(B, V))
    assert torch.equal(apart[1:].view(B, V), got)
