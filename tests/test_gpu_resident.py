"""GPU: sequences that run in one launch share the chip -- side by side where there is room, one after the other where
there is not, and without room for a while -- and give the results of a call that has the chip to itself."""
import threading
import time

import pytest

pytestmark = pytest.mark.gpu

SHARES = 8  # of the whole chip


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def amq():
    import paper_1802_00150_amd as m
    m.binding.lib()
    return m


@pytest.fixture
def held(amq):
    """held(shares): other launches of the kind keep that much of the chip until the test ends."""
    import torch
    taken = []

    def take(shares):
        taken.append(shares)
        amq.binding.debug_hold_sequence_shares(shares)
    yield take
    torch.cuda.synchronize()
    for n in taken:
        amq.binding.debug_hold_sequence_shares(-n)
    amq.binding.debug_set_sequence_spin_limit(0)
    torch.cuda.synchronize()


class Sequence:
    """One model with its inputs, and the sequence call on buffers of its own."""

    def __init__(self, amq, gates, I, H, B, k_w, k_a, steps):
        import torch
        self.amq, self.gates, self.I, self.H, self.B, self.k_w, self.k_a, self.steps = amq, gates, I, H, B, k_w, k_a, steps
        g = torch.Generator(device="cuda:0").manual_seed(I + 3 * H + 5 * B + gates)
        randn = lambda *s: torch.randn(*s, generator=g, device="cuda:0")  # noqa: E731
        self.d = [*amq.quantize_weights(randn(gates * H, I) * 0.05, k_w, 2),
                  *amq.quantize_weights(randn(gates * H, H) * 0.05, k_w, 2)]
        self.bias = randn(gates * H) * 0.1
        self.xs = randn(steps, B, I)
        self.h0, self.c0 = torch.tanh(randn(B, H)), randn(B, H)

    def workspace(self):
        make = self.amq.lstm_sequence_workspace if self.gates == 4 else self.amq.gru_sequence_workspace
        return make(self.I, self.H, self.B, self.k_a, self.xs.device)

    def run(self, ws):
        """Enqueues one call on the current stream: every h_t and the final state."""
        import torch
        h, c = self.h0.clone(), self.c0.clone()
        hs = torch.empty((self.steps, self.B, self.H), device=h.device)
        if self.gates == 4:
            self.amq.lstm_sequence(*self.d, self.I, self.H, self.bias, self.xs, h, c, self.k_a, 2, ws=ws, hs=hs)
        else:
            self.amq.gru_sequence(*self.d, self.I, self.H, self.bias, None, self.xs, h, self.k_a, 2, ws=ws, hs=hs)
        return hs, h, c


@pytest.mark.parametrize("gates,I,H,B,k_w,k_a", [(4, 300, 300, 16, 2, 2), (3, 130, 600, 33, 3, 2), (4, 1100, 300, 5, 2, 3)])
def test_without_room_the_piece_is_computed_alone(amq, held, gates, I, H, B, k_w, k_a):
    # the whole chip stays taken for longer than the launch may wait for room
    import torch
    s = Sequence(amq, gates, I, H, B, k_w, k_a, 4)
    ws = s.workspace()
    ref = s.run(ws)
    say("no room: gates=%d I=%d H=%d B=%d W%d/A%d" % (gates, I, H, B, k_w, k_a))
    held(SHARES)
    amq.binding.debug_set_sequence_spin_limit(1000)
    for got, want in zip(s.run(ws), ref):
        assert torch.equal(got, want)


def test_batch_1_without_room_goes_ahead(amq, held):
    import torch
    s = Sequence(amq, 4, 300, 300, 1, 2, 2, 70)
    ws = s.workspace()
    ref = s.run(ws)
    held(SHARES)
    amq.binding.debug_set_sequence_spin_limit(100000)
    got = s.run(ws)
    assert not amq.lstm_sequence_abandoned(ws, 300, 300, 1, 2)
    for g, w in zip(got, ref):
        assert torch.equal(g, w)


@pytest.mark.parametrize("H,B,k,share", [(300, 1, 2, 2), (300, 16, 2, 1), (1024, 64, 3, 8), (1024, 1, 3, 8), (600, 40, 2, 4)])
def test_a_claim_waits_only_where_there_is_no_room(amq, held, H, B, k, share):
    # share: ceil(workgroups / 32).  With the rest of the chip taken the call does not wait (it would for 0.2 s); and the
    # room it took is there again after it: the calls that follow find it too
    import torch
    s = Sequence(amq, 4, H, H, B, k, k, 3)
    ws = s.workspace()
    ref = s.run(ws)
    if share < SHARES:
        held(SHARES - share)
    torch.cuda.synchronize()
    start = time.perf_counter()
    for _ in range(3):
        got = s.run(ws)
    torch.cuda.synchronize()
    took = time.perf_counter() - start
    say("H=%d B=%d: %.2f ms" % (H, B, 1e3 * took))
    for g, w in zip(got, ref):
        assert torch.equal(g, w)
    assert took < 0.1


@pytest.mark.parametrize("shapes", [
    # small grids side by side, batch 1 and more
    [(4, 300, 300, 1, 2, 2, 70), (4, 300, 300, 16, 2, 2, 40), (3, 200, 400, 20, 2, 3, 40), (4, 650, 650, 1, 3, 3, 40)],
    # grids that take the whole chip, one after the other, among small ones
    [(4, 1024, 1024, 64, 3, 3, 12), (4, 1024, 1024, 1, 2, 2, 40), (3, 1024, 1024, 50, 2, 2, 12), (4, 300, 300, 16, 2, 2, 40)],
    # the forms that hold the most registers on (nearly) every compute unit: a launch that waits must not be in their way
    [(4, 2048, 2048, 17, 3, 2, 8), (4, 1500, 1500, 32, 3, 3, 8), (3, 1024, 1024, 64, 3, 2, 8), (4, 2048, 2048, 32, 2, 3, 8)],
])
def test_streams_and_threads_share_the_chip(amq, shapes):
    # every thread has a stream, a workspace and a model of its own and enqueues several calls without waiting
    import torch
    seqs = [Sequence(amq, *shape) for shape in shapes]
    refs = [s.run(s.workspace()) for s in seqs]
    torch.cuda.synchronize()
    results, errors, ready = [None] * len(seqs), [], threading.Barrier(len(seqs) + 1, timeout=60)

    def work(i):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                ws = seqs[i].workspace()
                results[i] = [seqs[i].run(ws)]  # (first calls allocate)
                stream.synchronize()
                ready.wait()
                results[i] += [seqs[i].run(ws) for _ in range(6)]
            stream.synchronize()
        except Exception as e:  # noqa: BLE001
            errors.append((i, repr(e)))

    say("shapes", shapes)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(seqs))]
    for t in threads:
        t.start()
    ready.wait()
    start = time.perf_counter()
    for t in threads:
        t.join()
    took = time.perf_counter() - start
    say("%.2f ms" % (1e3 * took))
    assert not errors, errors
    for i, ref in enumerate(refs):
        for call in results[i]:
            for g, w in zip(call, ref):
                assert torch.equal(g, w), (i, shapes[i])
    assert took < 0.2, "a launch waited until its time for room was up"


# word of the workspace of a batch-1 LSTM sequence behind its flag (amq_launch.h: kSeqGClaimed): the room that the launch took
CLAIMED = 1 + 256 // 4 + 1


def claimed(amq, s, ws):
    import torch
    torch.cuda.synchronize()
    off = int(amq.binding.lib().amq_lstm_sequence_flag_offset(s.I, s.H, 1, s.k_a))
    return int(ws[off:off + 4 * (CLAIMED + 1)].view(torch.int32)[CLAIMED])


def room(amq):
    """Full shares that are taken (light ones are counted from 256 on)."""
    import torch
    word = torch.full((1,), -1, dtype=torch.int32, device="cuda:0")
    amq.binding.debug_sequence_room(word)
    return int(word)


@pytest.mark.parametrize("gates,I,H,k_w,k_a", [(4, 128, 128, 2, 2), (4, 200, 160, 2, 3), (3, 300, 300, 2, 2), (4, 300, 300, 2, 2),
                                               (4, 1000, 224, 3, 3), (4, 448, 448, 2, 2), (3, 448, 449, 3, 2)])
def test_single_sequences_leave_room(amq, held, gates, I, H, k_w, k_a):
    # 2 to 29 workgroups: one share, alone on the chip (however many calls ran on that stream before) as beside another launch, and
    # it is given back
    import torch
    say("one share: gates=%d I=%d H=%d W%d/A%d" % (gates, I, H, k_w, k_a))
    s = Sequence(amq, gates, I, H, 1, k_w, k_a, 70)
    ws = s.workspace()
    alone = [s.run(ws) for _ in range(40)][-2:]
    assert gates != 4 or claimed(amq, s, ws) == 1
    assert room(amq) == 0
    held(SHARES - 1)
    beside = [s.run(ws) for _ in range(3)]
    assert gates != 4 or claimed(amq, s, ws) == 1  # (a call that waits in vain takes none)
    assert room(amq) == SHARES - 1
    for got in alone[1:] + beside:
        for g, w in zip(got, alone[0]):
            assert torch.equal(g, w)
