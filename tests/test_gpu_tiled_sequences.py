"""GPU: sequences of batches whose tiles take turns on a workgroup (amq_seqw_tiles.hip) against the same entries in batches that have a
workgroup for every tile, bit for bit; and what follows when a wait gives up."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amq():
    import paper_1802_00150_amd as m
    m.binding.lib()
    return m


def case(amq, gates, I, H, B, k_w, k_a, steps):
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(7 * I + 3 * H + B + gates + steps)
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda:0")  # noqa: E731
    d = [*amq.quantize_weights(randn(gates * H, I) * 0.05, k_w, 2), *amq.quantize_weights(randn(gates * H, H) * 0.05, k_w, 2)]
    bias = [randn(gates * H) * 0.1 for _ in range(2)]
    xs, h0, c0 = randn(steps, B, I), torch.tanh(randn(B, H)), randn(B, H)

    def run(lo, hi, T, hs=True):
        x, h, c = xs[:, lo:hi].contiguous(), h0[lo:hi].clone(), c0[lo:hi].clone()
        out = torch.full((steps, hi - lo, H), float("nan"), device=x.device) if hs else None
        if gates == 4:
            amq.lstm_sequence(*d, I, H, bias[0], x, h, c, k_a, T, hs=out)
        else:
            amq.gru_sequence(*d, I, H, *bias, x, h, k_a, T, hs=out)
        return [v for v in (out, h, c if gates == 4 else None) if v is not None]
    return run


# groups of 2 to 4 tiles, a last tile of 1 to 16 entries, groups of unequal numbers of tiles (one of a single tile), more entries than
# workgroups in a group and fewer, one and two stretches of 1024 entries, the fewest steps and several pieces; and shapes and
# numbers of steps next to those
@pytest.mark.parametrize("gates,I,H,B,k_w,k_a,steps", [
    (4, 1024, 1024, 65, 2, 2, 8), (4, 1024, 1024, 128, 3, 3, 9), (3, 1024, 1024, 256, 2, 3, 40), (4, 1000, 1008, 180, 2, 2, 7),
    (4, 2048, 2048, 33, 3, 2, 8), (4, 2048, 2048, 40, 2, 2, 8), (3, 2047, 2040, 97, 2, 2, 10), (3, 300, 2048, 128, 2, 2, 18),
    (4, 200, 260, 330, 2, 2, 14), (4, 129, 500, 200, 3, 3, 8), (3, 2048, 520, 161, 3, 2, 9), (4, 1025, 650, 112, 2, 2, 37),
    (4, 650, 650, 256, 3, 3, 11), (3, 1500, 1500, 48, 2, 2, 8), (4, 650, 1500, 96, 3, 2, 9), (4, 16, 650, 113, 2, 3, 8),
    (4, 300, 300, 256, 2, 3, 8), (4, 2048, 2048, 129, 2, 2, 8), (3, 800, 800, 512, 2, 2, 9),
    # two tiles on two stretches: 12 steps and fewer
    (4, 2048, 2048, 40, 2, 2, 12), (3, 1500, 1500, 48, 2, 2, 13), (4, 1100, 1300, 70, 2, 2, 11),
    # three tiles of 484, 517 and 532 workgroups per step, and of 495 with one entry of a step per workgroup
    (4, 700, 700, 176, 3, 3, 8), (3, 740, 740, 176, 2, 3, 8), (4, 606, 606, 224, 3, 2, 8), (3, 872, 872, 144, 2, 2, 8)])
def test_same_bits_as_batches_that_fit(amq, gates, I, H, B, k_w, k_a, steps):
    import torch
    for T in (2, 0):
        print("tiled", gates, I, H, B, k_w, k_a, steps, T, flush=True)
        run = case(amq, gates, I, H, B, k_w, k_a, steps)
        whole = run(0, B, T)
        again = run(0, B, T, hs=False)
        assert all(torch.equal(a, b) for a, b in zip(whole[1:], again))
        for lo in sorted({0, (B // 32) * 16, max(0, B - 20)}):
            hi = min(B, lo + 20)
            for w, p in zip(whole, run(lo, hi, T)):
                w = w[:, lo:hi] if w.dim() == 3 else w[lo:hi]
                assert bool(torch.isfinite(p).all()) and torch.equal(w, p), (lo, int((w != p).sum()))


@pytest.mark.parametrize("gates,H,B", [(4, 1024, 80), (3, 2048, 64)])
def test_gives_up_and_recovers(amq, gates, H, B):
    """With a wait that ends at its first failed poll the launch gives up, and the one behind it computes the piece."""
    import torch
    run = case(amq, gates, H, H, B, 2, 2, 8)
    want = run(0, B, 2)
    amq.binding.debug_set_sequence_spin_limit(1)
    try:
        got = run(0, B, 2)
        torch.cuda.synchronize()
    finally:
        amq.binding.debug_set_sequence_spin_limit(0)
    for w, g in zip(want, got):
        assert torch.equal(w, g)


def test_side_by_side_on_streams(amq):
    """Launches that want the whole chip, from several streams, with smaller ones between: each waits for its room.  With waits of
    sixteen times the usual length one that somebody is missing from takes over three seconds, far more than a slow host."""
    import time

    import torch
    shapes = [(4, 1024, 1024, 128, 2, 2, 16), (3, 650, 650, 192, 2, 3, 16), (4, 300, 300, 16, 2, 2, 16), (4, 2048, 2048, 64, 2, 2, 16)]
    runs = [case(amq, *s) for s in shapes]
    want = [r(0, s[3], 2) for r, s in zip(runs, shapes)]
    streams = [torch.cuda.Stream() for _ in shapes]

    def round_of_calls():
        got = []
        for r, s, q in zip(runs, shapes, streams):
            with torch.cuda.stream(q):
                got.append(r(0, s[3], 2))
        return got
    round_of_calls()  # (first calls on a stream allocate)
    torch.cuda.synchronize()
    amq.binding.debug_set_sequence_spin_limit(1 << 23)
    try:
        start = time.perf_counter()
        got = [round_of_calls() for _ in range(3)]
        torch.cuda.synchronize()
        took = time.perf_counter() - start
    finally:
        amq.binding.debug_set_sequence_spin_limit(0)
    print("%.2f ms" % (1e3 * took), flush=True)
    assert took < 1.0, "somebody waited for room that was there"
    for one in got:
        for w, g in zip(want, one):
            assert all(torch.equal(a, b) for a, b in zip(w, g))
