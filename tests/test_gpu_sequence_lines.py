"""GPU: sequences in one launch at the lines between their forms -- how long the first poll waits, and which waves gather the codes
(amq_seqw.hip, amq_seq1_body.h) -- against per-step calls, bit for bit.  The word in which such a launch says how it ended is
read as well: the workspace is filled with a pattern first, so that per-step launches in its place, a wait that gave up or a launch
without room would show."""
import pytest

pytestmark = pytest.mark.gpu

FILL = 0xA5
ENDED, GAVE_UP = 0, 1


@pytest.fixture(scope="module")
def amq():
    import paper_1802_00150_amd as m
    m.binding.lib()
    return m


def last_bytes(H, B, k_a):
    """Bytes of what a batched sequence's launch keeps at the end of the workspace, its word first."""
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    wpr = 4 * ((H + 127) // 128)
    entry = (k_a * (wpr + 1) + 15) // 16 * 16
    return up(256 + up(16 * B * H) + up(16 * ((B + 15) // 16) * 16 * entry) + 2 * up(4 * B * H))


def same_bits_as_steps(amq, gates, I, H, B, k_w, k_a, steps=4):
    """Runs the sequence and the steps; returns the word of the launch (None for a single entry)."""
    import torch
    print("lines", gates, I, H, B, k_w, k_a, flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(I + 3 * H + 5 * B + gates)
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda:0")  # noqa: E731
    d = [*amq.quantize_weights(randn(gates * H, I) * 0.05, k_w, 2), *amq.quantize_weights(randn(gates * H, H) * 0.05, k_w, 2)]
    bias = [randn(gates * H) * 0.1 for _ in range(2)]
    xs, h, c = randn(steps, B, I), torch.tanh(randn(B, H)), randn(B, H)
    hs = torch.full((steps, B, H), float("nan"), device=h.device)
    hq, cq = h.clone(), c.clone()
    ws = (amq.lstm_sequence_workspace if gates == 4 else amq.gru_sequence_workspace)(I, H, B, k_a, h.device).fill_(FILL)
    if gates == 4:
        amq.lstm_sequence(*d, I, H, bias[0], xs, hq, cq, k_a, 2, ws=ws, hs=hs)
    else:
        amq.gru_sequence(*d, I, H, *bias, xs, hq, k_a, 2, ws=ws, hs=hs)
    word = None
    if B > 1:
        at = ws.numel() - last_bytes(H, B, k_a)
        word = int(ws[at:at + 4].view(torch.int32).item())
    for t in range(steps):
        if gates == 4:
            h, c = amq.lstm_step(*d, I, H, bias[0], xs[t], h, c, k_a, 2)
        else:
            h = amq.gru_step(*d, I, H, *bias, xs[t], h, k_a, 2)
        assert bool(torch.isfinite(h).all()) and torch.equal(hs[t], h), (t, int((hs[t] != h).sum()))
    assert torch.equal(hq, h) and (gates == 3 or torch.equal(cq, c))
    return word


# one workgroup per tile, one with several entries, eight and nine of them; long inputs
@pytest.mark.parametrize("gates,I,H,B,k_w,k_a", [
    (4, 8, 8, 2, 2, 2), (3, 20, 20, 33, 3, 1), (4, 128, 128, 5, 2, 2), (3, 129, 129, 5, 2, 3), (4, 600, 112, 16, 1, 2), (3, 1024, 130, 17, 3, 3)])
def test_few_workgroups(amq, gates, I, H, B, k_w, k_a):
    assert same_bits_as_steps(amq, gates, I, H, B, k_w, k_a) == ENDED


# the longest states that ask at once and the shortest that wait: 192 units of an LSTM, 128 of a GRU; LSTMs of six plane products up to 256.
# LSTMs against the form that captured streams take, which adds in the same order
@pytest.mark.parametrize("gates,H,k_w,k_a", [
    (4, 40, 2, 2), (4, 192, 2, 2), (4, 193, 2, 2), (3, 128, 2, 2), (3, 129, 3, 3), (4, 256, 2, 3), (4, 257, 2, 3), (4, 200, 3, 2), (3, 100, 3, 2)])
def test_single_entries(amq, gates, H, k_w, k_a):
    import torch
    I, steps = H + 30, 70
    if gates == 3:
        assert same_bits_as_steps(amq, gates, I, H, 1, k_w, k_a, steps) is None
        return
    print("lines", gates, I, H, 1, k_w, k_a, flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(H)
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda:0")  # noqa: E731
    d = [*amq.quantize_weights(randn(4 * H, I) * 0.05, k_w, 2), *amq.quantize_weights(randn(4 * H, H) * 0.05, k_w, 2)]
    bias, xs, h0, c0 = randn(4 * H) * 0.1, randn(steps, 1, I), torch.tanh(randn(1, H)), randn(1, H)
    h, c, hs = h0.clone(), c0.clone(), torch.full((steps, 1, H), float("nan"), device=h0.device)
    ws = amq.lstm_sequence_workspace(I, H, 1, k_a, h.device).fill_(FILL)

    def call():
        amq.lstm_sequence(*d, I, H, bias, xs, h, c, k_a, 2, ws=ws, hs=hs)

    call()
    assert not amq.lstm_sequence_abandoned(ws, I, H, 1, k_a)
    got = [t.clone() for t in (hs, h, c)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(2):
        h.copy_(h0)
        c.copy_(c0)
        hs.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(got, (hs, h, c)):
            assert bool(torch.isfinite(b).all()) and torch.equal(a, b)


# either side of 256 and 1024 units and of inputs of 1536 for every number of weight planes; a GRU's nine plane products with inputs of
# one and of two stretches
@pytest.mark.parametrize("gates,I,H,B,k_w,k_a", [
    (4, 1537, 256, 9, 1, 2), (3, 1537, 257, 9, 1, 1), (4, 1536, 256, 9, 2, 2), (3, 1100, 257, 17, 2, 3), (4, 1537, 1024, 5, 2, 2), (4, 1537, 1025, 5, 2, 3),
    (4, 1500, 1024, 16, 3, 3), (4, 1500, 1025, 16, 3, 2), (4, 1537, 1025, 4, 3, 1), (3, 1024, 1030, 18, 3, 3), (3, 1025, 1030, 18, 3, 3),
    (3, 1536, 1500, 2, 3, 3)])
def test_who_gathers(amq, gates, I, H, B, k_w, k_a):
    assert same_bits_as_steps(amq, gates, I, H, B, k_w, k_a) == ENDED


# one or both kinds of wave gather, with and without a shared contraction, which has two barriers more: with waits that end at their second
# poll the launch gives up, all waves leave, and the piece is computed alone
@pytest.mark.parametrize("gates,I,H,B,k_w,k_a", [
    (4, 300, 1024, 18, 2, 2), (4, 1500, 1500, 18, 2, 2), (3, 1100, 1300, 3, 3, 3), (4, 600, 1100, 16, 3, 3), (4, 2000, 1024, 18, 2, 2),
    (4, 2000, 1100, 18, 3, 3), (3, 1700, 1030, 5, 3, 2)])
def test_gives_up(amq, gates, I, H, B, k_w, k_a):
    amq.binding.debug_set_sequence_spin_limit(1)
    try:
        assert same_bits_as_steps(amq, gates, I, H, B, k_w, k_a) == GAVE_UP
    finally:
        amq.binding.debug_set_sequence_spin_limit(0)


# lengths on both sides of every half of 512 positions that the shared contraction splits at, by which launch they were computed
@pytest.mark.parametrize("gates,I,H,B,k_w,k_a", [
    (4, 1025, 1025, 2, 2, 2), (4, 64, 1536, 17, 2, 2), (3, 2048, 1537, 5, 2, 2), (4, 2048, 2048, 16, 3, 3), (4, 2047, 2047, 3, 1, 1),
    (3, 1030, 1281, 18, 1, 2), (4, 700, 1500, 20, 1, 3), (3, 1536, 1536, 2, 2, 1), (4, 33, 1100, 3, 3, 3), (4, 1537, 1537, 8, 3, 2)])
def test_long_states_take_one_launch(amq, gates, I, H, B, k_w, k_a):
    assert same_bits_as_steps(amq, gates, I, H, B, k_w, k_a) == ENDED
