"""The work a user of this library has it do, as cases that can be timed and compared.

Every case goes through the package's public entry points (paper_1802_00150_amd) on inputs that already lie
in GPU memory, with the quantized weights, workspace and output buffers that a serving or scoring program
keeps between calls.  Kinds of case:

  matvec     on-line quantization of a batch of vectors, then the binary product (the quantity of Table 6)
  lstm_step  one LSTM step per call, state carried by the caller (step-by-step serving)
  gru_step   one GRU step per call, then the quantized output projection of its h_t
  lstm_seq   a whole LSTM sequence with given inputs in one call
  gru_seq    a whole GRU sequence with given inputs in one call
  lm_step    token -> distribution, one step per call (generation)
  lm_seq     a token sequence -> every distribution in one call (teacher forcing)
  lm_score   log-probability of given next words of token sequences (perplexity)
  quantize   off-line quantization of a weight matrix (packed planes + per-row coefficients)
  train      training side: forward pass through the quantized weights and straight-through backward pass

Shapes and value distributions are those of `inputs.py` and of the tests, and generic ones around them:
hidden sizes 200 to 2048, vocabularies 2000 to 42000, batches 1 to 256, 1 to 4 bits.
"""
import math

import torch

import paper_1802_00150_amd as amq

T = 2  # alternating cycles, as everywhere in the paper


def listed():
    return [
        # Table 6's unit of work at batch 1: quantize the activation, one 4096 x 1024 product.  The smallest call.
        dict(name="matvec_4096x1024_b1", kind="matvec", m=4096, n=1024, B=1, k_w=2, k_a=2),
        # The output projection of many hidden states at once (10K vocabulary, W2/A3).
        dict(name="matvec_10000x1024_b1024", kind="matvec", m=10000, n=1024, B=1024, k_w=2, k_a=3),
        # Step-by-step serving of a few concurrent sequences; sizes that fit no tile.
        dict(name="lstm_step_650_b13", kind="lstm_step", I=650, H=650, B=13, k_w=2, k_a=2),
        # The small language model's recurrence (hidden 300), one sequence of 35 steps.
        dict(name="lstm_seq_300_b1", kind="lstm_seq", I=300, H=300, B=1, k_w=2, k_a=2, steps=35),
        # The benchmark's headline: hidden 1024, 64 concurrent sequences, W3/A3.
        dict(name="lstm_seq_1024_b64", kind="lstm_seq", I=1024, H=1024, B=64, k_w=3, k_a=3, steps=35),
        # A larger hidden size than the tuned ones, ragged in every direction.
        dict(name="lstm_seq_1500_b20", kind="lstm_seq", I=1500, H=1500, B=20, k_w=2, k_a=2, steps=35),
        # GRU with a large batch and its quantized output projection, step by step.
        dict(name="gru_step_1024_b256", kind="gru_step", I=1024, H=1024, B=256, V=10000, k_w=2, k_a=2, k_as=3),
        # Generation: one token in, one distribution over the large vocabulary out.
        dict(name="lm_step_1024_v42000_b1", kind="lm_step", E=1024, H=1024, V=42000, B=1, k_w=2, k_a=2, k_as=2),
        # Teacher forcing with every distribution wanted, a medium model with the 10K vocabulary.
        dict(name="lm_seq_650_v10000_b20", kind="lm_seq", E=650, H=650, V=10000, B=20, k_w=2, k_a=2, k_as=3, steps=35),
        # Scoring a corpus with the large model (the quantity behind the perplexities).  The largest case.
        dict(name="lm_score_1024_v42000_b64", kind="lm_score", E=1024, H=1024, V=42000, B=64, k_w=2, k_a=2, k_as=2, steps=35),
        # Off-line quantization of a large matrix with heavy tails.
        dict(name="quantize_16384x4096_k2", kind="quantize", rows=16384, cols=4096, k=2),
        # Training: forward through the quantized gate matrix of the large model and backward, 3 bits.
        dict(name="train_4096x2048_k3", kind="train", rows=4096, cols=2048, k=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges, no larger than the largest listed one."""
    most = {m: max(work(c)[m] for c in listed()) for m in ("bytes", "flops")}
    while True:
        kind = rng.choice(["matvec", "lstm_step", "gru_step", "lstm_seq", "gru_seq", "lm_step", "lm_seq", "lm_score",
                           "quantize", "train"])
        k_w, k_a = rng.choice([(2, 2), (2, 2), (3, 3), (2, 3)])
        H = _log(rng, 200, 2048)
        I = rng.choice([H, _log(rng, 200, 2048)])
        B = rng.choice([1, _log(rng, 2, 256)])
        V = _log(rng, 2000, 42000)
        steps = rng.randint(10, 70)
        if kind == "matvec":
            c = dict(kind=kind, m=_log(rng, 600, 42000), n=_log(rng, 200, 4096), B=rng.choice([1, _log(rng, 2, 1024)]),
                     k_w=k_w, k_a=k_a)
        elif kind == "lstm_step":
            c = dict(kind=kind, I=I, H=H, B=B, k_w=k_w, k_a=k_a)
        elif kind == "gru_step":
            c = dict(kind=kind, I=I, H=H, B=B, V=V, k_w=k_w, k_a=k_a, k_as=3)
        elif kind in ("lstm_seq", "gru_seq"):
            c = dict(kind=kind, I=I, H=H, B=B, k_w=k_w, k_a=k_a, steps=steps)
        elif kind == "lm_step":
            c = dict(kind=kind, E=I, H=H, V=V, B=B, k_w=k_w, k_a=k_a, k_as=k_a)
        elif kind in ("lm_seq", "lm_score"):
            c = dict(kind=kind, E=I, H=H, V=V, B=B, k_w=k_w, k_a=k_a, k_as=k_a, steps=steps)
        else:
            c = dict(kind=kind, rows=_log(rng, 1000, 42000), cols=_log(rng, 200, 4096), k=rng.choice([1, 2, 2, 3, 3, 4]))
        w = work(c)
        if all(w[m] <= most[m] for m in most):
            return c


# ------------------------------------------------------------------------------------------ inputs


class _Draws:
    """Seeded normal and integer tensors on the GPU."""

    def __init__(self, seed):
        self.dev = torch.device("cuda")
        self.g = torch.Generator(device=self.dev).manual_seed(180200150 + int(seed))

    def normal(self, shape, std):
        return torch.randn(shape, generator=self.g, device=self.dev) * std

    def ids(self, shape, hi):
        return torch.randint(0, hi, shape, generator=self.g, device=self.dev, dtype=torch.int64)

    def hidden(self, shape):
        """Values like those of a running recurrence: inside (-1, 1)."""
        return torch.tanh(self.normal(shape, 0.5))


def _cell_weights(d, gates, I, H, k_w):
    std = 0.05 if H <= 512 else 0.02
    Wxp, ax = amq.quantize_weights(d.normal((gates * H, I), std), k_w, T)
    Whp, ah = amq.quantize_weights(d.normal((gates * H, H), std), k_w, T)
    return Wxp, ax, Whp, ah


def prepare(case, seed):
    c, d = case, _Draws(seed)
    kind = c["kind"]
    s = dict(case=c)
    if kind == "matvec":
        s["W"] = amq.quantize_weights(d.normal((c["m"], c["n"]), 0.02), c["k_w"], T)
        s["x"] = d.normal((c["B"], c["n"]), 1.0)
    elif kind in ("lstm_step", "gru_step"):
        I, H, B = c["I"], c["H"], c["B"]
        gates = 4 if kind == "lstm_step" else 3
        s["cell"] = _cell_weights(d, gates, I, H, c["k_w"])
        s["bias"] = [d.normal((gates * H,), 0.1) for _ in range(1 if kind == "lstm_step" else 2)]
        s["x"], s["h"], s["c"] = d.normal((B, I), 1.0), d.hidden((B, H)), d.normal((B, H), 0.5)
        s["h_out"], s["c_out"] = torch.empty_like(s["h"]), torch.empty_like(s["c"])
        if kind == "lstm_step":
            s["ws"] = amq.lstm_workspace(I, H, B, c["k_a"], d.dev)
        else:
            s["ws"] = amq.gru_workspace(I, H, B, c["k_a"], d.dev)
            s["proj"] = amq.quantize_weights(d.normal((c["V"], H), 0.02), c["k_w"], T)
    elif kind in ("lstm_seq", "gru_seq"):
        I, H, B = c["I"], c["H"], c["B"]
        gates = 4 if kind == "lstm_seq" else 3
        s["cell"] = _cell_weights(d, gates, I, H, c["k_w"])
        s["xs"] = d.normal((c["steps"], B, I), 0.1 if B == 1 else 1.0)
        s["state"] = torch.empty((2, B, H), device=d.dev)
        s["hs"] = torch.empty((c["steps"], B, H), device=d.dev)
        make = amq.lstm_sequence_workspace if kind == "lstm_seq" else amq.gru_sequence_workspace
        s["ws"] = make(I, H, B, c["k_a"], d.dev)
    elif kind in ("lm_step", "lm_seq", "lm_score"):
        E, H, V, B = c["E"], c["H"], c["V"], c["B"]
        s["emb"] = amq.quantize_weights(d.normal((V, E), 0.1), c["k_a"], T)
        s["cell"] = _cell_weights(d, 4, E, H, c["k_w"])
        s["soft"] = amq.quantize_weights(d.normal((V, H), 0.02), c["k_w"], T)
        s["bias_s"] = d.normal((V,), 0.1)
        if kind == "lm_step":
            s["ids"] = d.ids((B,), V)
            s["state"] = torch.stack([d.hidden((B, H)), d.normal((B, H), 0.5)])  # h and c, updated in place by every step
            s["ws"] = amq.lm_workspace(E, H, V, B, c["k_a"], c["k_as"], d.dev)
            s["out"] = torch.empty((B, V), device=d.dev)
        else:
            L = amq.binding.lib()
            query = L.amq_lm_sequence_workspace_bytes if kind == "lm_seq" else L.amq_lm_sequence_score_workspace_bytes
            nbytes = int(query(E, H, V, B, c["k_a"], c["k_as"]))
            s["ids"] = d.ids((c["steps"], B), V)
            s["targets"] = d.ids((c["steps"], B), V)
            s["state"] = torch.empty((2, B, H), device=d.dev)
            s["ws"] = torch.empty(nbytes, dtype=torch.uint8, device=d.dev)
            s["out"] = torch.empty((c["steps"], B, V) if kind == "lm_seq" else (c["steps"], B), device=d.dev)
    else:
        W = d.normal((c["rows"], c["cols"]), 0.02)
        if kind == "quantize":  # heavy tails: one entry in a hundred ten times larger
            tail = torch.rand(W.shape, generator=d.g, device=d.dev) < 0.01
            W = torch.where(tail, W * 10.0, W)
            s["W"] = W.contiguous()
        else:
            s["W"] = W.requires_grad_(True)
            s["grad"] = d.normal((c["rows"], c["cols"]), 1e-3)
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "matvec":
        planes, beta = amq.quantize_activations(s["x"], c["k_a"], T)
        Y = amq.binary_gemm(*s["W"], c["n"], planes, beta)
        return dict(planes=planes, beta=beta, Y=Y)
    if kind == "lstm_step":
        h, cc = amq.lstm_step(*s["cell"], c["I"], c["H"], s["bias"][0], s["x"], s["h"], s["c"], c["k_a"], T, ws=s["ws"],
                              h_out=s["h_out"], c_out=s["c_out"])
        return dict(h=h, c=cc)
    if kind == "gru_step":
        h = amq.gru_step(*s["cell"], c["I"], c["H"], *s["bias"], s["x"], s["h"], c["k_a"], T, ws=s["ws"],
                         h_out=s["h_out"])
        planes, beta = amq.quantize_activations(h, c["k_as"], T)
        return dict(h=h, logits=amq.binary_gemm(*s["proj"], c["H"], planes, beta))
    if kind == "lstm_seq":
        s["state"].zero_()
        h, cc = amq.lstm_sequence(*s["cell"], c["I"], c["H"], None, s["xs"], s["state"][0], s["state"][1], c["k_a"], T,
                                  ws=s["ws"], hs=s["hs"])
        return dict(h=h, c=cc, hs=s["hs"])
    if kind == "gru_seq":
        s["state"].zero_()
        h = amq.gru_sequence(*s["cell"], c["I"], c["H"], None, None, s["xs"], s["state"][0], c["k_a"], T, ws=s["ws"],
                             hs=s["hs"])
        return dict(h=h, hs=s["hs"])
    if kind == "lm_step":
        y = amq.lm_step(*s["emb"], c["E"], *s["cell"], c["H"], None, *s["soft"], s["bias_s"], s["ids"], s["state"][0],
                        s["state"][1], c["k_a"], c["k_as"], T, ws=s["ws"], logprob=s["out"])
        return dict(logprob=y, state=s["state"])
    if kind == "lm_seq":
        s["state"].zero_()
        y = amq.lm_sequence(*s["emb"], c["E"], *s["cell"], c["H"], None, *s["soft"], s["bias_s"], s["ids"],
                            s["state"][0], s["state"][1], c["k_a"], c["k_as"], T, ws=s["ws"], logprob=s["out"])
        return dict(logprob=y, state=s["state"])
    if kind == "lm_score":
        s["state"].zero_()
        y = amq.lm_sequence_score(*s["emb"], c["E"], *s["cell"], c["H"], None, *s["soft"], s["bias_s"], s["ids"],
                                  s["targets"], s["state"][0], s["state"][1], c["k_a"], c["k_as"], T, ws=s["ws"],
                                  out=s["out"])
        return dict(logprob=y, state=s["state"])
    if kind == "quantize":
        planes, alpha = amq.quantize_weights(s["W"], c["k"], T)
        return dict(planes=planes, alpha=alpha)
    s["W"].grad = None
    w_hat = amq.fake_quantize(s["W"], c["k"], T)
    w_hat.backward(s["grad"])
    return dict(w_hat=w_hat.detach(), grad=s["W"].grad)


# ------------------------------------------------------------------------------------------ what a pass needs


def _packed(rows, n, k):
    """Bytes of a k-bit row-wise quantization: planes and coefficients."""
    return rows * (k * n / 8.0 + 4.0 * k)


def work(case):
    """Bytes: every weight, input and state read once, every output written once.  Operations: a product counts
    2 m n B (what the equivalent dense product of the reconstructed operands needs, however many bit planes the
    kernels multiply), a quantization the method's own 2 T k^2 + 2 (T + 1) k per entry."""
    c = case
    kind = c["kind"]
    ops = lambda k: 2 * T * k * k + 2 * (T + 1) * k  # noqa: E731
    if kind in ("quantize", "train"):
        n = float(c["rows"]) * c["cols"]
        if kind == "quantize":
            return dict(bytes=4 * n + _packed(c["rows"], c["cols"], c["k"]), flops=ops(c["k"]) * n)
        return dict(bytes=4 * n * 4, flops=ops(c["k"]) * n)  # W and the gradient in, w_hat and W.grad out
    if kind == "matvec":
        m, n, B = c["m"], c["n"], c["B"]
        return dict(bytes=_packed(m, n, c["k_w"]) + 4.0 * B * n + _packed(B, n, c["k_a"]) + 4.0 * B * m,
                    flops=2.0 * m * n * B + ops(c["k_a"]) * B * n)
    H, B = c["H"], c["B"]
    I = c.get("I", c.get("E"))
    gates = 3 if kind.startswith("gru") else 4
    steps = c.get("steps", 1)
    cell_bytes = _packed(gates * H, I, c["k_w"]) + _packed(gates * H, H, c["k_w"])
    state = 4.0 * B * H * (2 if gates == 4 else 1)
    flops = steps * (2.0 * gates * H * (I + H) * B + ops(c["k_a"]) * B * H)
    if kind in ("lstm_step", "gru_step"):
        nbytes = cell_bytes + 4.0 * B * I + 2 * state
        flops += ops(c["k_a"]) * B * I
        if kind == "gru_step":
            nbytes += _packed(c["V"], H, c["k_w"]) + 4.0 * B * c["V"]
            flops += 2.0 * c["V"] * H * B + ops(c["k_as"]) * B * H
        return dict(bytes=nbytes, flops=flops)
    if kind in ("lstm_seq", "gru_seq"):
        return dict(bytes=cell_bytes + 4.0 * steps * B * (I + H) + 2 * state, flops=flops + steps * ops(c["k_a"]) * B * I)
    V = c["V"]
    rows = steps * B
    out = 4.0 * rows * V if kind != "lm_score" else 12.0 * rows
    nbytes = cell_bytes + 2 * state + _packed(rows, I, c["k_a"]) + 8.0 * rows + _packed(V, H, c["k_w"]) + 4.0 * V + out
    return dict(bytes=nbytes, flops=flops + 2.0 * V * H * rows + ops(c["k_as"]) * rows * H)


def tolerance(case):
    """Sums of 32-bit values: 1e-5.  Whole words of packed codes may differ where an entry lies within rounding of
    a midpoint.  In a recurrence such a near-tie moves one quantized entry of one row of h by the distance of two
    neighbouring codes, and what follows in that row with it: about 1e-2 of that row, 1e-3 over a batch."""
    if case["kind"] in ("lstm_seq", "gru_seq", "lm_seq", "lm_score"):
        return {"rel": 1e-3}
    if case["kind"] in ("quantize", "matvec"):
        return {"rel": 1e-5, "differ": 1e-5}
    return {"rel": 1e-5}
