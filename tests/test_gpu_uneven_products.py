"""GPU: large products on 32 x 32 tiles whose row blocks do not come out even over the waves of a workgroup (amq_mfma32_body.h),
at vectors of 769 .. 1024 entries around the lines of the dispatch: outputs, and the log-softmax and scores that are formed with
them, against dense binary64 products of the reconstructed operands."""
import pytest

from gpu_util import host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amq():
    import paper_1802_00150_amd as m
    m.binding.lib()
    return m


def operands(amq, m, n, B, k_w, k_a):
    import torch
    print("uneven product %d x %d batch %d W%d/A%d" % (m, n, B, k_w, k_a), flush=True)
    g = torch.Generator(device="cuda").manual_seed(m + n + B)
    W = amq.quantize_weights(torch.randn((m, n), generator=g, device="cuda") * 0.05, k_w, 2)
    x = torch.randn((B, n), generator=g, device="cuda")
    bias = torch.randn((m,), generator=g, device="cuda")
    X = amq.quantize_activations(x, k_a, 2)
    ref = amq.dequantize(*X, n).double() @ amq.dequantize(*W, n).double().t().contiguous() + bias.double()
    return W, x, X, bias, ref


# row blocks per workgroup: 1, 2, 5, 9 (one wave has two), 10, 11, 23; the last workgroup short; groups of columns short
@pytest.mark.parametrize("m,n,B,k_w,k_a", [(35233, 1000, 17, 2, 3), (35168, 1024, 31, 2, 3), (10000, 1024, 256, 2, 3),
                                           (9200, 770, 255, 2, 3), (42000, 800, 65, 3, 3), (11000, 1024, 270, 3, 3),
                                           (5001, 1024, 600, 3, 2), (3001, 300, 1000, 2, 2),
                                           # either side of the lines that the padding of columns and the rounding of
                                           # blocks draw: batch 48, a full batch and one more, 13 blocks in rounds of 4
                                           (42000, 900, 48, 2, 3), (42000, 900, 49, 2, 3), (16000, 1024, 128, 3, 2),
                                           (16000, 1024, 129, 3, 2), (10000, 1024, 300, 3, 3), (10000, 1024, 384, 3, 3),
                                           # columns of Y that begin at any multiple of four bytes
                                           (9997, 1024, 400, 3, 3), (9998, 800, 300, 2, 3), (9999, 1500, 65, 2, 2)])
def test_outputs(amq, m, n, B, k_w, k_a):
    W, _, X, bias, ref = operands(amq, m, n, B, k_w, k_a)
    tol = 1e-4 * ref.abs() + 1e-4 * ref.pow(2).mean(1, keepdim=True).sqrt()
    Y = amq.binary_gemm(*W, n, *X, bias=bias)
    assert bool(((Y.double() - ref).abs() <= tol).all())


@pytest.mark.parametrize("V,H,B,k_w,k_a", [(35233, 1000, 17, 2, 3), (10000, 1024, 256, 2, 3), (42000, 800, 65, 3, 3)])
def test_log_softmax_of_them(amq, V, H, B, k_w, k_a):
    import torch
    W, x, _, bias, ref = operands(amq, V, H, B, k_w, k_a)
    want = torch.log_softmax(ref, dim=1)
    got = amq.softmax_layer(*W, H, bias, x, k_a, 2)
    tol = 1e-4 * want.abs() + 1e-4 * want.pow(2).mean(1, keepdim=True).sqrt()
    assert bool(((got.double() - want).abs() <= tol).all())
    assert host(got).shape == (B, V)
