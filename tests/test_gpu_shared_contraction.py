"""GPU: resident sequences whose vectors are longer than 1024 entries, where two waves share the contraction of a row block
(amq_seqw.hip), against per-step calls, bit for bit: the partial sums are integers of at most 1024, which binary32 holds, so nothing may
be lost.  And inputs on either side of 1536 entries, where the gather of the codes by one or by both of the two waves changes with the
weights' bits and the state's length."""
import pytest

pytestmark = pytest.mark.gpu


# either side of 2, 3 and 4 halves of 512 positions, ragged last words; the longer block on either side; every number of planes
# that shares, one that does not; a batch of one tile and a part of a second
@pytest.mark.parametrize("gates,I,H,B,k_w,k_a", [
    (4, 1025, 1025, 2, 2, 2), (4, 64, 1536, 17, 2, 2), (3, 2048, 1537, 5, 2, 2), (4, 2048, 2048, 16, 3, 3), (3, 1100, 1024, 20, 3, 3),
    (4, 1300, 513, 4, 2, 2), (4, 2047, 2047, 3, 1, 1), (3, 1030, 1281, 18, 1, 2), (4, 700, 1500, 20, 1, 3), (3, 1536, 1536, 2, 2, 1),
    (4, 33, 1100, 3, 3, 3), (4, 1025, 1600, 3, 2, 3),
    (4, 1536, 1200, 9, 2, 2), (4, 1537, 1200, 9, 2, 2), (4, 1537, 1537, 8, 3, 2), (3, 1537, 1537, 7, 2, 3), (4, 2000, 300, 24, 2, 2),
    (3, 1600, 40, 9, 3, 3), (4, 300, 24, 16, 2, 2), (3, 100, 1000, 8, 1, 3)])
def test_same_bits_as_steps(gates, I, H, B, k_w, k_a):
    import torch
    import paper_1802_00150_amd as amq
    print("shared", gates, I, H, B, k_w, k_a, flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(I + 3 * H + B + gates)
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda:0")  # noqa: E731
    d = [*amq.quantize_weights(randn(gates * H, I) * 0.05, k_w, 2), *amq.quantize_weights(randn(gates * H, H) * 0.05, k_w, 2)]
    # the largest sums there are: a row of weights and an entry of the state with all signs alike
    d[0][:, 0], d[2][:, 0] = 0, 0
    bias = [randn(gates * H) * 0.1 for _ in range(2)]
    steps = 3
    xs, h, c = randn(steps, B, I), torch.tanh(randn(B, H)), randn(B, H)
    h[0] = -h[0].abs()
    hs = torch.full((steps, B, H), float("nan"), device=h.device)
    hq, cq = h.clone(), c.clone()
    if gates == 4:
        amq.lstm_sequence(*d, I, H, bias[0], xs, hq, cq, k_a, 2, hs=hs)
    else:
        amq.gru_sequence(*d, I, H, *bias, xs, hq, k_a, 2, hs=hs)
    for t in range(steps):
        if gates == 4:
            h, c = amq.lstm_step(*d, I, H, bias[0], xs[t], h, c, k_a, 2)
        else:
            h = amq.gru_step(*d, I, H, *bias, xs[t], h, k_a, 2)
        assert bool(torch.isfinite(h).all()) and torch.equal(hs[t], h), (t, int((hs[t] != h).sum()))
    assert torch.equal(hq, h) and (gates == 3 or torch.equal(cq, c))
