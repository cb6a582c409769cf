"""GPU: the split recurrent step (front and back launch, amq_step.hip) -- what sequences take whose grid does not fit the
chip as a whole, and all batched ones on a stream that is being captured.  Every shape here is checked to have gone that
way, by the pieces of the workspace it left its marks in."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_vec_close, host, to_dev
from test_gpu_lm import lm_gpu_step, lm_oracle_step, lm_setup

pytestmark = pytest.mark.gpu

MARK = 0xA5


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


def up256(n):
    return (n + 255) // 256 * 256


def route(ws, off, I, H, B, k_a):
    """Which form of the recurrence wrote to a marked workspace, whose regions after those of a single step start at byte
    `off`: two sets of input codes and coefficients and the x-side sums (split step), then the resident kernel's, which
    end with its copies of the initial state (ws ends there)."""
    wpr = 4 * ((I + 127) // 128)
    own = 2 * (up256(4 * k_a * B * wpr) + up256(4 * B * k_a)) + 16 * B * H  # (a single step stores no sums)
    touched = lambda a, n: bool((ws[a:a + n] != MARK).any().item())  # noqa: E731
    split = touched(off, own)
    resident = touched(ws.numel() - 2 * up256(4 * B * H), 2 * up256(4 * B * H))
    assert not (split and resident)
    return "split" if split else "resident" if resident else "steps"


class Sequence:
    def __init__(self, amq, gates, I, H, B, k_w, k_a, steps):
        import torch
        self.amq, self.gates, self.I, self.H, self.B, self.k_a, self.steps = amq, gates, I, H, B, k_a, steps
        g = np.random.default_rng(I + 3 * H + 7 * B + gates)
        f32 = lambda *s: g.standard_normal(s).astype(np.float32)  # noqa: E731
        self.w = [*oracle.quantize_rows(f32(gates * H, I) * np.float32(0.05), k_w, 2),
                  *oracle.quantize_rows(f32(gates * H, H) * np.float32(0.05), k_w, 2)]
        self.bias = [f32(gates * H) * np.float32(0.1) for _ in range(2)]
        self.xs, self.h0, self.c0 = f32(steps, B, I), np.tanh(f32(B, H)), f32(B, H)
        self.d = [to_dev(t) for t in self.w]
        self.dbias = [to_dev(t) for t in self.bias]
        self.dxs, self.dh, self.dc = to_dev(self.xs), to_dev(self.h0), to_dev(self.c0)
        self.hs = torch.empty((steps, B, H), device="cuda:0")
        make = amq.lstm_sequence_workspace if gates == 4 else amq.gru_sequence_workspace
        self.ws = make(I, H, B, k_a, "cuda:0")

    def call(self, ws=None):
        ws = self.ws if ws is None else ws
        if self.gates == 4:
            self.amq.lstm_sequence(*self.d, self.I, self.H, self.dbias[0], self.dxs, self.dh, self.dc, self.k_a, 2, ws=ws,
                                   hs=self.hs)
        else:
            self.amq.gru_sequence(*self.d, self.I, self.H, *self.dbias, self.dxs, self.dh, self.k_a, 2, ws=ws, hs=self.hs)

    def restart(self):
        self.dh.copy_(to_dev(self.h0))
        self.dc.copy_(to_dev(self.c0))

    def route(self):
        L = self.amq.binding.lib()
        off = (L.amq_lstm_workspace_bytes if self.gates == 4 else L.amq_gru_workspace_bytes)(self.I, self.H, self.B, self.k_a)
        return route(self.ws, off, self.I, self.H, self.B, self.k_a)

    def per_step(self):
        """(h_t, c_t) of every step by the per-step call."""
        h, c, out = to_dev(self.h0), to_dev(self.c0), []
        for t in range(self.steps):
            if self.gates == 4:
                h, c = self.amq.lstm_step(*self.d, self.I, self.H, self.dbias[0], self.dxs[t], h, c, self.k_a, 2)
            else:
                h = self.amq.gru_step(*self.d, self.I, self.H, *self.dbias, self.dxs[t], h, self.k_a, 2)
            out.append((h, c))
        return out

    def oracle_step(self, t, h, c):
        """The oracle's step t on a given previous state."""
        if self.gates == 4:
            return oracle.lstm_step(*self.w, self.I, self.H, self.bias[0], self.xs[t], h, c, self.k_a, 2)
        return oracle.gru_step(*self.w, self.I, self.H, *self.bias, self.xs[t], h, self.k_a, 2), c


# more than 256 workgroups of 16 units and 16 entries; vectors of at most 1024 entries and (two stretches, 8 slots per
# lane of the quantizer) beyond, blocks of unequal length, ragged tiles and units, 1 to 3 bits, one and two steps
SHAPES = [(1024, 1024, 70, 2, 2, 4), (300, 1021, 65, 3, 3, 3), (1024, 513, 128, 1, 3, 3), (130, 1024, 100, 2, 1, 1),
          (1500, 1500, 33, 2, 2, 4), (1100, 1030, 65, 3, 3, 3), (2048, 2048, 40, 2, 3, 3), (300, 1500, 50, 3, 2, 2),
          (2000, 700, 90, 1, 2, 3), (1030, 1024, 80, 3, 1, 2)]


@pytest.mark.parametrize("gates", [4, 3])
@pytest.mark.parametrize("I,H,B,k_w,k_a,steps", SHAPES)
def test_sequences_beyond_the_chip(amq, gates, I, H, B, k_w, k_a, steps):
    # every h_t and the final state equal those of the per-step calls bit for bit; each step agrees with the oracle's on
    # the same previous state
    import torch
    say("split gates=%d I=%d H=%d B=%d W%d/A%d steps=%d" % (gates, I, H, B, k_w, k_a, steps))
    s = Sequence(amq, gates, I, H, B, k_w, k_a, steps)
    s.ws.fill_(MARK)
    s.call()
    assert s.route() == "split"
    ref = s.per_step()
    for t in range(steps):
        assert torch.equal(s.hs[t], ref[t][0]), "h_%d" % (t + 1)
    assert torch.equal(s.dh, ref[-1][0])
    if gates == 4:
        assert torch.equal(s.dc, ref[-1][1])
    for t in sorted({0, steps - 1}):
        h, c = (s.h0, s.c0) if t == 0 else (host(ref[t - 1][0]), host(ref[t - 1][1]))
        h_ref, c_ref = s.oracle_step(t, h, c)
        assert_vec_close(host(s.hs[t]), h_ref, "h_%d" % (t + 1))
        assert_vec_close(host(ref[t][1]) if gates == 4 else c, c_ref, "c_%d" % (t + 1))


@pytest.mark.parametrize("gates,I,H,B,k_w,k_a,steps", [(4, 300, 200, 17, 3, 3, 5), (3, 200, 300, 40, 2, 2, 4),
                                                       (4, 1100, 130, 20, 2, 3, 3), (3, 130, 1100, 5, 3, 2, 3)])
def test_captured_sequences(amq, gates, I, H, B, k_w, k_a, steps):
    # shapes that take the resident kernel elsewhere take the split step on a captured stream, with the same results; every
    # replay is compared, with eager calls between
    import torch
    say("captured gates=%d I=%d H=%d B=%d W%d/A%d" % (gates, I, H, B, k_w, k_a))
    s = Sequence(amq, gates, I, H, B, k_w, k_a, steps)
    s.ws.fill_(MARK)
    s.call()
    assert s.route() == "resident"
    ref = [s.hs.clone(), s.dh.clone(), s.dc.clone()]
    for t, (h, _) in enumerate(s.per_step()):
        assert torch.equal(s.hs[t], h)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        s.call()
    other = torch.empty_like(s.ws)
    for replay in range(3):
        s.restart()
        s.hs.fill_(float("nan"))
        s.ws.fill_(MARK)
        graph.replay()
        for got, want in zip((s.hs, s.dh, s.dc), ref):
            assert torch.equal(got, want), replay
        assert s.route() == "split"
        s.restart()
        s.call(ws=other)
        torch.cuda.synchronize()


def test_captured_batch_1_sequence(amq):
    # the one-launch recurrence of batch 1 in a graph: each replay claims its room and gives it back
    import time

    import torch
    s = Sequence(amq, 4, 300, 300, 1, 2, 2, 70)
    s.call()
    ref = [s.hs.clone(), s.dh.clone(), s.dc.clone()]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        s.call()
    other = torch.empty_like(s.ws)
    for replay in range(3):
        s.restart()
        s.hs.fill_(float("nan"))
        graph.replay()
        for got, want in zip((s.hs, s.dh, s.dc), ref):
            assert torch.equal(got, want), replay
        s.restart()
        torch.cuda.synchronize()
        start = time.perf_counter()
        s.call(ws=other)
        torch.cuda.synchronize()
        assert time.perf_counter() - start < 0.1, "no room was left"


@pytest.mark.parametrize("E,H,V,B,k,steps", [(1024, 1024, 130, 70, 2, 3), (300, 1021, 555, 65, 3, 2), (1100, 1500, 200, 33, 2, 3),
                                             (1030, 1024, 97, 80, 3, 2)])
def test_language_model_sequences_beyond_the_chip(amq, E, H, V, B, k, steps):
    # the inputs looked up a step ahead by the front launch: state equal to that of step-by-step calls, log-probabilities
    # (all of them, and those of given words) against the oracle on the GPU's own state
    import torch
    from paper_1802_00150_amd import inputs
    say("split lm E=%d H=%d V=%d B=%d k=%d" % (E, H, V, B, k))
    cfg = inputs.language_model(trial=E + B, steps=steps, B=B, H=H, E=E, vocab=V, k=k)
    q = lm_setup(cfg, k)
    dq = {n: to_dev(q[n]) for n in ("Ep", "ae", "Wxp", "ax", "Whp", "ah", "Wsp", "as", "bias", "bs")}
    model = (dq["Ep"], dq["ae"], E, dq["Wxp"], dq["ax"], dq["Whp"], dq["ah"], H, dq["bias"], dq["Wsp"], dq["as"], dq["bs"])
    ids = torch.from_numpy(np.ascontiguousarray(cfg["ids"])).to("cuda:0")
    targets = np.random.default_rng(B).integers(0, V, size=(steps, B)).astype(np.int64)
    sh, sc = torch.zeros((B, H), device="cuda:0"), torch.zeros((B, H), device="cuda:0")
    states = [(host(sh), host(sc))]
    for t in range(steps):
        lm_gpu_step(amq, q, dq, cfg["ids"][t], sh, sc, k, k)
        states.append((host(sh), host(sc)))
    L = amq.binding.lib()
    n = int(L.amq_lm_sequence_workspace_bytes(E, H, V, B, k, k))
    ws = torch.full((n,), MARK, dtype=torch.uint8, device="cuda:0")
    dh, dc = torch.zeros((B, H), device="cuda:0"), torch.zeros((B, H), device="cuda:0")
    lp = host(amq.lm_sequence(*model, ids, dh, dc, k, k, 2, ws=ws))
    rows = 4096 // B * B
    off = int(L.amq_lstm_workspace_bytes(E, H, B, k)) + up256(4 * rows * H) + int(L.amq_softmax_layer_workspace_bytes(V, H, rows, k))
    assert route(ws, off, E, H, B, k) == "split"
    assert torch.equal(dh, sh) and torch.equal(dc, sc)
    dh.zero_(), dc.zero_()
    score = host(amq.lm_sequence_score(*model, ids, torch.from_numpy(targets).to("cuda:0"), dh, dc, k, k, 2))
    assert torch.equal(dh, sh) and torch.equal(dc, sc)
    for t in range(steps):
        h1, c1, ref = lm_oracle_step(q, cfg["ids"][t], *states[t], k)
        assert_vec_close(states[t + 1][0], h1, "h step %d" % t)
        assert_vec_close(states[t + 1][1], c1, "c step %d" % t)
        # (the output layer on the GPU's own h_t: the oracle's differs in the last digits, which may move a code)
        _, ref = oracle.softmax_layer(q["Wsp"], q["as"], H, q["bs"], states[t + 1][0], k, 2)
        assert_vec_close(lp[t], ref, "logprob step %d" % t)
        want = ref[np.arange(B), targets[t]].astype(np.float64)
        tol = 1e-4 * np.abs(want) + 1e-4 * np.log(V)   # as the full log-probabilities: their r.m.s. is about log V
        assert (np.abs(score[t] - want) <= tol).all()
