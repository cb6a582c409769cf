"""GPU: batch-1 sequences in one launch per piece (amq_seq1_body.h) against the forms they replace -- the per-step calls, and
for LSTMs with vectors of at most 1024 entries the form that captured streams take -- bit for bit, at the edges of its slots
and lanes; and what follows when a wait gives up."""
import numpy as np
import pytest

from gpu_util import assert_vec_close, host

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def amq():
    import paper_1802_00150_amd as m
    m.binding.lib()
    return m


class Model:
    def __init__(self, amq, gates, I, H, k_w, k_a, steps, T=2):
        import torch
        self.amq, self.gates, self.I, self.H, self.k_w, self.k_a, self.steps, self.T = amq, gates, I, H, k_w, k_a, steps, T
        g = torch.Generator(device="cuda:0").manual_seed(7 * I + 3 * H + gates + steps)
        randn = lambda *s: torch.randn(*s, generator=g, device="cuda:0")  # noqa: E731
        self.d = [*amq.quantize_weights(randn(gates * H, I) * 0.05, k_w, 2),
                  *amq.quantize_weights(randn(gates * H, H) * 0.05, k_w, 2)]
        self.bias = [randn(gates * H) * 0.1 for _ in range(2)]
        self.xs = randn(steps, 1, I)
        self.h0, self.c0 = torch.tanh(randn(1, H)), randn(1, H)
        make = amq.lstm_sequence_workspace if gates == 4 else amq.gru_sequence_workspace
        self.ws = make(I, H, 1, k_a, self.xs.device)
        self.ws.fill_(0xA5)

    def start(self):
        import torch
        self.h, self.c = self.h0.clone(), self.c0.clone()
        self.hs = torch.full((self.steps, 1, self.H), float("nan"), device=self.h.device)

    def call(self, hs=True, ws=None):
        ws = self.ws if ws is None else ws
        if self.gates == 4:
            self.amq.lstm_sequence(*self.d, self.I, self.H, self.bias[0], self.xs, self.h, self.c, self.k_a, self.T, ws=ws,
                                   hs=self.hs if hs else None)
        else:
            self.amq.gru_sequence(*self.d, self.I, self.H, *self.bias, self.xs, self.h, self.k_a, self.T, ws=ws,
                                  hs=self.hs if hs else None)

    def result(self):
        return [t.clone() for t in ((self.hs, self.h, self.c) if self.gates == 4 else (self.hs, self.h))]

    def per_step(self):
        import torch
        h, c, hs = self.h0.clone(), self.c0.clone(), []
        for t in range(self.steps):
            if self.gates == 4:
                h, c = self.amq.lstm_step(*self.d, self.I, self.H, self.bias[0], self.xs[t], h, c, self.k_a, self.T)
            else:
                h = self.amq.gru_step(*self.d, self.I, self.H, *self.bias, self.xs[t], h, self.k_a, self.T)
            hs.append(h.clone())
        return [torch.stack(hs), h, c][:3 if self.gates == 4 else 2]

    def captured(self):
        import torch
        self.start()
        self.call()  # (first calls allocate)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            self.call()
        self.start_in_place()
        graph.replay()
        torch.cuda.synchronize()
        return self.result()

    def start_in_place(self):
        self.h.copy_(self.h0)
        self.c.copy_(self.c0)
        self.hs.fill_(float("nan"))


SHAPES = [  # (I, H): one unit, less than a slot, edges of slots and of the forms, unequal blocks on either side of 1024
    (64, 1), (40, 63), (130, 64), (100, 65), (256, 192), (300, 256), (33, 257), (300, 300), (384, 320), (321, 321), (500, 384),
    (512, 448), (1024, 449), (650, 512), (100, 513), (650, 650), (129, 768), (1000, 769), (1024, 1024), (1025, 130), (2048, 512),
    (1100, 700), (200, 1025), (1500, 1280), (1300, 1281), (1536, 1536), (1, 1537), (1900, 1792), (2048, 1793), (2048, 2048)]


@pytest.mark.parametrize("gates", [4, 3])
@pytest.mark.parametrize("I,H", SHAPES)
def test_equal_to_the_forms_it_replaces(amq, gates, I, H):
    import torch
    k_w, k_a = [(2, 2), (3, 3), (2, 3), (3, 2)][(I + H) % 4]
    m = Model(amq, gates, I, H, k_w, k_a, 5)
    say("single gates=%d I=%d H=%d W%d/A%d" % (gates, I, H, k_w, k_a))
    ref = m.captured() if gates == 4 and max(I, H) <= 1024 else m.per_step()
    m.ws.fill_(0xA5)
    m.start()
    m.call()
    for got, want in zip(m.result(), ref):
        assert torch.equal(got, want)
    m.start()
    m.call(hs=False)
    assert torch.equal(m.h, ref[1])


@pytest.mark.parametrize("gates,I,H,k,steps,T", [(4, 300, 300, 2, 1, 2), (3, 300, 300, 2, 1, 2), (4, 1100, 200, 3, 1, 2),
                                                 (3, 700, 700, 3, 65, 2), (4, 1030, 1030, 2, 130, 2), (3, 90, 90, 2, 3, 0),
                                                 (4, 1200, 90, 3, 3, 1), (3, 520, 600, 3, 3, 4)])
def test_pieces_single_steps_and_cycles(amq, gates, I, H, k, steps, T):
    # a single step (the state is read by waves that another may have overtaken), several pieces, other numbers of cycles
    import torch
    m = Model(amq, gates, I, H, k, k, steps, T)
    say("single gates=%d I=%d H=%d k=%d steps=%d T=%d" % (gates, I, H, k, steps, T))
    ref = m.captured() if gates == 4 and max(I, H) <= 1024 else m.per_step()
    for _ in range(5):
        m.start()
        m.call()
        for got, want in zip(m.result(), ref):
            assert torch.equal(got, want)


@pytest.mark.parametrize("gates,I,H,k", [(3, 300, 300, 2), (4, 1100, 300, 3), (3, 130, 1300, 2)])
def test_a_piece_whose_waits_give_up_is_computed_again(amq, gates, I, H, k):
    # shapes without a word that tells the caller: the launch that follows computes the piece alone (sums in another order:
    # a unit in the last place of binary32 per step, far below what moves a code in so few steps), and clears the flag
    import torch
    m = Model(amq, gates, I, H, k, k, 4)
    m.start()
    m.call()
    ref = [host(t) for t in m.result()]
    say("gives up: gates=%d I=%d H=%d k=%d" % (gates, I, H, k))
    amq.binding.debug_set_sequence_spin_limit(1)
    try:
        m.start()
        m.call()
        torch.cuda.synchronize()
    finally:
        amq.binding.debug_set_sequence_spin_limit(0)
    got = [host(t) for t in m.result()]
    for t in range(4):
        assert_vec_close(got[0][t], ref[0][t], "h_%d" % (t + 1))
    for g, w in zip(got[1:], ref[1:]):
        assert_vec_close(g, w, "state")
    if gates == 4:
        assert not amq.lstm_sequence_abandoned(m.ws, I, H, 1, k)
    assert np.isfinite(got[0]).all()
    m.start()
    m.call()
    for g, w in zip(m.result(), ref):
        assert np.array_equal(host(g), w)


@pytest.mark.parametrize("gates,I,H,k", [(3, 2048, 2048, 2), (3, 300, 2000, 3), (4, 2048, 2048, 3)])
def test_recovers_from_a_state_that_is_all_saved(amq, gates, I, H, k):
    # beside a launch that holds all but a few compute units: the workgroups that fit give up, those that arrive when it has
    # ended find the flag raised and leave at once, and the launch that follows must find the state of them all.  (Nothing in
    # the workspace is left from an earlier call.)
    import time

    import torch
    m = Model(amq, gates, I, H, k, k, 4)
    m.start()
    m.call()
    ref = [host(t) for t in m.result()]
    holder = Model(amq, 4, 960, 960, 2, 2, 64)  # 60 workgroups x 4 tiles
    holder.xs, holder.ws = torch.randn(64, 64, 960, device="cuda:0"), amq.lstm_sequence_workspace(960, 960, 64, 2, "cuda:0")
    holder.h0, holder.c0 = torch.zeros(64, 960, device="cuda:0"), torch.zeros(64, 960, device="cuda:0")
    side = torch.cuda.Stream()
    say("late workgroups: gates=%d I=%d H=%d k=%d" % (gates, I, H, k))
    for _ in range(3):
        m.start()
        m.ws.fill_(0xA5)
        holder.start()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            holder.call(hs=False)
        time.sleep(1e-4)
        amq.binding.debug_set_sequence_spin_limit(1)
        try:
            m.call()
            torch.cuda.synchronize()
        finally:
            amq.binding.debug_set_sequence_spin_limit(0)
        got = [host(t) for t in m.result()]
        for t in range(4):  # (few steps: sums in another order, as above)
            assert_vec_close(got[0][t], ref[0][t], "h_%d" % (t + 1))
        for g, w in zip(got[1:], ref[1:]):
            assert_vec_close(g, w, "state")


@pytest.mark.parametrize("captured", [False, True])
@pytest.mark.parametrize("I,H,hs", [(300, 300, True), (700, 1024, True), (1024, 1024, False)])
def test_a_piece_that_is_given_up_leaves_the_state_as_it_was(amq, I, H, hs, captured):
    # in the last step the first to look find nothing and give up, while the last ones find all of it there and finish
    import torch
    m = Model(amq, 4, I, H, 2, 2, 2)
    m.start()
    m.call(hs)
    ref = m.result()
    graph = torch.cuda.CUDAGraph() if captured else None
    say("given up: I=%d H=%d hs=%s captured=%s" % (I, H, hs, captured))
    amq.binding.debug_set_sequence_spin_limit(1)
    try:
        torch.cuda.synchronize()
        if captured:
            with torch.cuda.graph(graph):
                m.call(hs)
        seen = 0
        for _ in range(20):
            m.start_in_place()
            graph.replay() if captured else m.call(hs)
            torch.cuda.synchronize()
            gave_up = amq.lstm_sequence_abandoned(m.ws, I, H, 1, 2)
            seen += gave_up
            want = (torch.full_like(m.hs, float("nan")), m.h0, m.c0) if gave_up else ref
            for got, w in list(zip(m.result(), want))[0 if hs else 1:]:
                assert torch.equal(got.nan_to_num(7.0), w.nan_to_num(7.0))
    finally:
        amq.binding.debug_set_sequence_spin_limit(0)
    say("%d of 20" % seen)
    assert seen > 0


def test_small_workspace_and_other_codes_take_the_steps(amq):
    # a GRU workspace without the regions of the one-launch form, and code widths it does not take
    import torch
    m = Model(amq, 3, 200, 200, 2, 2, 3)
    ref = m.per_step()
    m.start()
    m.call(ws=amq.gru_workspace(200, 200, 1, 2, m.xs.device))
    for got, want in zip(m.result(), ref):
        assert torch.equal(got, want)
    m = Model(amq, 3, 200, 200, 1, 4, 3)
    ref = m.per_step()
    m.start()
    m.call()
    for got, want in zip(m.result(), ref):
        assert torch.equal(got, want)
