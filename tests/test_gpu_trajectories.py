"""GPU: long free-running sequences of small batches with vectors above 1024 entries against the oracle.

The matrix-core kernels that take these shapes sum exact integers and apply the coefficients once; the oracle sums in
binary64.  Their h_t agree to the last digits, and in a free-running sequence such a digit can move an entry that lies at
a midpoint of the code table: from there on that row of the batch follows another trajectory, which is as good.  So every
step is compared with the oracle's on the GPU's own previous state, and the two trajectories row by row up to the first
code that moved, which has to be shown to lie at a midpoint."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_vec_close, host, to_dev

pytestmark = pytest.mark.gpu

T = 2


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def amq():
    import paper_1802_00150_amd as m
    m.binding.lib()
    return m


@pytest.fixture(autouse=True)
def threads():
    oracle.set_threads(oracle.host_threads())
    yield
    oracle.set_threads(1)


def moved_codes(a, b, k):
    """Entries of two versions of one vector that the quantizer tells apart at the first stage where it does (the greedy
    codes, then those of each cycle), and their distance from what decides there on version b, in units of the largest
    code value.  None: the same codes at every stage."""
    (ca, aa), (cb, ab) = oracle.greedy(a, k), oracle.greedy(b, k)
    scale = np.abs(oracle.code_table(ab)[0]).max()
    r = b.astype(np.float32).copy()
    for i in range(k):   # plane by plane: the sign of the residual
        diff = ca[i] != cb[i]
        if diff.any():
            return np.nonzero(diff)[0], np.abs(r[diff]) / scale
        r = r - np.where(cb[i] == 1, ab[i], -ab[i]).astype(np.float32)
    for _ in range(T):
        aa, ab = oracle.ls(a, ca, aa)[0], oracle.ls(b, cb, ab)[0]
        v, _, mid = oracle.code_table(ab)
        ca, cb = oracle.bst(a, aa), oracle.bst(b, ab)
        diff = (ca != cb).any(axis=0)
        if diff.any():
            return np.nonzero(diff)[0], np.abs(mid[None, :].astype(np.float64) - b[diff][:, None]).min(axis=1) / np.abs(v).max()
    return None


def test_moved_codes_finds_the_entry_and_its_distance():
    g = np.random.default_rng(3)
    b = g.standard_normal(400).astype(np.float32)
    assert moved_codes(b, b, 2) is None
    code, alpha = oracle.greedy(b, 2)
    alpha = oracle.ls(b, code, alpha)[0]
    mid = oracle.code_table(alpha)[2]
    e = int(np.abs(b - mid[2]).argmin())
    a = b.copy()
    a[e] = mid[2] + (mid[2] - b[e])   # to the other side
    entries, distance = moved_codes(a, b, 2)
    assert entries.tolist() == [e] and abs(distance[0] - abs(b[e] - mid[2]) / np.abs(oracle.code_table(alpha)[0]).max()) < 1e-6


@pytest.mark.parametrize("gates,I,H,B,k_w,k_a,steps,seed", [
    (4, 1500, 1500, 8, 3, 3, 70, 0), (4, 1500, 1500, 8, 3, 3, 70, 1), (4, 1500, 1500, 8, 3, 3, 70, 2),
    (4, 1600, 1700, 4, 2, 2, 70, 0), (4, 1600, 1700, 4, 2, 2, 70, 1), (4, 300, 1100, 16, 2, 3, 70, 0),
    (4, 2048, 1030, 2, 3, 3, 35, 0), (3, 1500, 1500, 8, 3, 3, 70, 0), (3, 1030, 2048, 5, 2, 2, 35, 0)])
def test_small_batches_of_long_vectors(amq, gates, I, H, B, k_w, k_a, steps, seed):
    import torch
    g = np.random.default_rng(1000 * seed + I + 3 * H + B + gates)
    f32 = lambda *s: g.standard_normal(s).astype(np.float32)  # noqa: E731
    w = [*oracle.quantize_rows(f32(gates * H, I) * np.float32(0.02), k_w, T),
         *oracle.quantize_rows(f32(gates * H, H) * np.float32(0.02), k_w, T)]
    xs = f32(steps, B, I)
    d, dxs = [to_dev(t) for t in w], to_dev(xs)
    say("trajectory gates=%d I=%d H=%d B=%d W%d/A%d seed=%d" % (gates, I, H, B, k_w, k_a, seed))

    def oracle_step(t, h, c):
        if gates == 4:
            return oracle.lstm_step(*w, I, H, None, xs[t], h, c, k_a, T)
        return oracle.gru_step(*w, I, H, None, None, xs[t], h, k_a, T), c

    dh, dc = (torch.zeros((B, H), device="cuda:0") for _ in range(2))
    hs = torch.empty((steps, B, H), device="cuda:0")
    if gates == 4:
        amq.lstm_sequence(*d, I, H, None, dxs, dh, dc, k_a, T, hs=hs)
    else:
        amq.gru_sequence(*d, I, H, None, None, dxs, dh, k_a, T, hs=hs)
    gh, gc = (torch.zeros((B, H), device="cuda:0") for _ in range(2))
    h, c = np.zeros((B, H), np.float32), np.zeros((B, H), np.float32)   # the oracle's trajectory
    parted, worst = {}, 0.0   # rows whose codes have moved: step, entries, distance
    for t in range(steps):
        before = host(gh), host(gc)
        if gates == 4:
            gh, gc = amq.lstm_step(*d, I, H, None, dxs[t], gh, gc, k_a, T)
        else:
            gh = amq.gru_step(*d, I, H, None, None, dxs[t], gh, k_a, T)
        assert torch.equal(gh, hs[t]), "h_%d of the sequence call differs from the per-step call's" % (t + 1)
        h_own, c_own = oracle_step(t, *before)
        assert_vec_close(host(gh), h_own, "h_%d against the oracle on the GPU's own state" % (t + 1))
        if gates == 4:
            assert_vec_close(host(gc), c_own, "c_%d against the oracle on the GPU's own state" % (t + 1))
        h, c = oracle_step(t, h, c)
        now = host(gh)
        rows = [b for b in range(B) if b not in parted]
        assert_vec_close(now[rows], h[rows], "h_%d of the rows no code of which has moved" % (t + 1))
        worst = max(worst, float(np.abs(now[rows] - h[rows]).max() / np.sqrt((h[rows].astype(np.float64) ** 2).mean())))
        for b in rows:
            moved = moved_codes(now[b], h[b], k_a)
            if moved is not None:
                entries, distance = moved
                assert (distance <= 1e-5).all(), "row %d step %d: entries %s moved, %s from a midpoint" % (b, t + 1, entries, distance)
                parted[b] = (t + 1, len(entries), float(distance.max()))
        if len(parted) == B:
            break
    if parted:
        rows = list(parted)
        apart = np.linalg.norm(now[rows] - h[rows], axis=1) / np.linalg.norm(h[rows], axis=1)
        say("  rows that parted (step, moved entries, distance from a midpoint): %s; apart by %s at the end" % (parted, apart))
    say("  largest difference of the other rows, in units of the r.m.s. of h: %.2g" % worst)
    assert len(parted) <= B // 2
