"""GPU: recurrent steps of small batches in one launch (amq_step_once.hip).  Steps whose state is updated in place take two launches
and the same arithmetic: the two agree bit for bit, also where every wait gives up and the workgroups quantize for themselves, on
several streams whose launches take every slot several times, when tags come round, and in a replayed graph.  Which form a step took is
read from the library's count."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amq():
    import paper_1802_00150_amd as m
    m.binding.lib()
    return m


class Step:
    def __init__(self, amq, gates, I, H, B, k_w, k_a, seed=0):
        import torch
        print("step in one launch gates=%d I=%d H=%d B=%d W%d/A%d" % (gates, I, H, B, k_w, k_a), flush=True)
        g = torch.Generator(device="cuda:0").manual_seed(I + 3 * H + B + seed)
        randn = lambda *s: torch.randn(*s, generator=g, device="cuda:0")  # noqa: E731
        self.amq, self.gates, self.args, self.k_a, self.T = amq, gates, (I, H), k_a, 2
        self.d = [*amq.quantize_weights(randn(gates * H, I) * 0.04, k_w, 2), *amq.quantize_weights(randn(gates * H, H) * 0.04, k_w, 2)]
        self.bias = [randn(gates * H) * 0.1 for _ in range(1 if gates == 4 else 2)]
        self.x, self.h, self.c = randn(B, I), torch.tanh(randn(B, H)), randn(B, H)
        self.ws = (amq.lstm_workspace if gates == 4 else amq.gru_workspace)(I, H, B, k_a, "cuda:0")

    def into(self, h, h_out, c, c_out):
        if self.gates == 4:
            self.amq.lstm_step(*self.d, *self.args, *self.bias, self.x, h, c, self.k_a, self.T, ws=self.ws, h_out=h_out, c_out=c_out)
            return h_out, c_out
        self.amq.gru_step(*self.d, *self.args, *self.bias, self.x, h, self.k_a, self.T, ws=self.ws, h_out=h_out)
        return (h_out,)

    def two_launches(self):
        h, c = self.h.clone(), self.c.clone()
        return self.into(h, h, c, c)

    def once(self):
        import torch
        return self.into(self.h, torch.full_like(self.h, -7.0), self.c, torch.full_like(self.c, -7.0))


def launched_once(amq, call):
    """Result of the call, and whether it was issued as one launch."""
    before = amq.binding.debug_one_launch_steps()
    got = call()
    return got, amq.binding.debug_one_launch_steps() - before == 1


def same(a, b):
    import torch
    return all(torch.equal(p, q) for p, q in zip(a, b))


# one launch: one entry more and fewer than a tile, ragged units and vectors, one and two stretches, blocks of unequal stretches, the
# most workgroups that still take this path (56 of 256, up to four entries 96, with vectors of up to 512 entries 88 and W3/A2 120) ...
ONCE = [(300, 300, 2, 2, 2), (650, 650, 13, 2, 2), (1, 300, 17, 2, 2), (2048, 333, 16, 3, 2), (701, 650, 15, 3, 2),
        (129, 1030, 4, 2, 2), (1024, 1024, 4, 3, 2), (1500, 1500, 2, 3, 2), (33, 1, 7, 2, 2),
        (512, 512, 24, 2, 2), (256, 256, 56, 3, 2), (200, 201, 48, 3, 3), (512, 512, 4, 3, 3)]
# ... and two: one workgroup more, other numbers of bits, larger batches
TWICE = [(701, 650, 16, 3, 2), (1024, 1024, 5, 2, 2), (1536, 1537, 2, 2, 2), (512, 512, 25, 2, 2), (256, 257, 56, 3, 2), (513, 300, 25, 2, 2),
         (300, 300, 4, 2, 3), (513, 512, 4, 3, 3), (512, 512, 25, 3, 3), (1, 1030, 17, 2, 3), (128, 1024, 16, 2, 2), (700, 701, 33, 3, 2), (1500, 1500, 20, 2, 2),
         (2048, 2048, 5, 3, 3), (2000, 333, 31, 3, 3), (1024, 1024, 48, 2, 3), (1024, 1024, 64, 3, 3)]


@pytest.mark.parametrize("gates", [4, 3])
@pytest.mark.parametrize("I,H,B,k_w,k_a", ONCE + TWICE)
def test_same_as_two_launches(amq, gates, I, H, B, k_w, k_a):
    s = Step(amq, gates, I, H, B, k_w, k_a)
    want, one = launched_once(amq, s.two_launches)
    assert not one
    for _ in range(3):
        got, one = launched_once(amq, s.once)
        assert one == ((I, H, B, k_w, k_a) in ONCE) and same(got, want)
    # every wait gives up: the codes are looked for where they never are
    amq.binding.debug_set_sequence_spin_limit(1)
    try:
        got, one = launched_once(amq, s.once)
    finally:
        amq.binding.debug_set_sequence_spin_limit(0)
    assert one == ((I, H, B, k_w, k_a) in ONCE) and same(got, want)


@pytest.mark.parametrize("T,k,once", [(0, 2, True), (4, 2, True), (5, 2, False), (60, 2, False), (2, 3, True), (3, 3, False)])
def test_many_cycles_take_two_launches(amq, T, k, once):
    # one launch would be slower, and from about 40 cycles on much slower: its waits are shorter than the quantizer takes
    s = Step(amq, 4, 300, 300, 7, k, k)
    s.T = T
    got, one = launched_once(amq, s.once)
    assert one == once and same(got, s.two_launches())


def test_streams_and_slots(amq):
    import torch
    steps = [Step(amq, 4, 300, 300, 7, 2, 2), Step(amq, 3, 650, 650, 14, 3, 2), Step(amq, 4, 1100, 1024, 4, 2, 2)]
    want = [s.two_launches() for s in steps]
    streams = [torch.cuda.Stream() for _ in steps]
    torch.cuda.synchronize()
    got, before = [], amq.binding.debug_one_launch_steps()
    for _ in range(40):
        for i, s in enumerate(steps):
            with torch.cuda.stream(streams[i]):
                got.append((i, s.once()))
    torch.cuda.synchronize()
    assert amq.binding.debug_one_launch_steps() - before == len(got) > 3 * 32  # (slots)
    assert all(same(g, want[i]) for i, g in got)


def test_tags_come_round(amq):
    # after 2^32 launches a tag is used again, in the same slot; what the launch before left there under that tag is not taken for the
    # codes of this one (the counter is set past the launches in between)
    import torch
    s = Step(amq, 4, 1500, 1500, 2, 2, 2)
    hook, first = amq.binding.debug_one_launch_steps, 77
    before = hook()
    try:
        hook(first)
        for _ in range(16):
            s.once()
        hook(1 << 30)
        Step(amq, 4, 300, 300, 2, 2, 2).once()
        s.x, s.h = s.x.flip(1).contiguous(), s.h.flip(1).contiguous()
        want = s.two_launches()
        hook(first)
        got = [s.once() for _ in range(16)]
        torch.cuda.synchronize()
    finally:
        hook(before + (1 << 20))
    assert [same(g, want) for g in got] == [True] * 16


def test_graph_replays(amq):
    import torch
    s = Step(amq, 4, 300, 300, 7, 2, 2)
    want = s.two_launches()
    h, c = torch.empty_like(s.h), torch.empty_like(s.c)
    graph = torch.cuda.CUDAGraph()
    before = amq.binding.debug_one_launch_steps()
    with torch.cuda.graph(graph):
        s.into(s.h, h, s.c, c)
    assert amq.binding.debug_one_launch_steps() == before  # (a captured tag would come back at every replay)
    for _ in range(3):
        h.fill_(-7.0), c.fill_(-7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert same((h, c), want)
        x = s.x.clone()
        s.x.copy_(x.flip(0))  # other inputs in the same place
        graph.replay()
        torch.cuda.synchronize()
        assert same((h, c), s.two_launches())
        s.x.copy_(x)


def test_null_stream_beside_a_captured_one(amq):
    # whether the null stream is being captured cannot be asked while a blocking stream is: steps and sequences run all the same
    import ctypes
    import torch
    s = Step(amq, 4, 300, 300, 7, 2, 2)
    want = s.two_launches()
    xs, ws = s.x.repeat(5, 1, 1), amq.lstm_sequence_workspace(300, 300, 7, 2, "cuda:0")

    def sequence(h, c):
        amq.lstm_sequence(*s.d, *s.args, *s.bias, xs, h, c, 2, 2, ws=ws)
        return h, c
    seq = sequence(s.h.clone(), s.c.clone())
    hip, stream = ctypes.CDLL("libamdhip64.so"), ctypes.c_void_p()
    assert hip.hipStreamCreate(ctypes.byref(stream)) == 0
    x, h, c = torch.zeros(16, device="cuda:0"), torch.empty_like(s.h), torch.empty_like(s.c)
    state = s.h.clone(), s.c.clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(torch.cuda.ExternalStream(stream.value)):
        graph.capture_begin(capture_error_mode="relaxed")
        try:
            x.add_(1)
            with torch.cuda.stream(torch.cuda.default_stream()):
                s.into(s.h, h, s.c, c)
                got = sequence(*state)
        finally:
            graph.capture_end()
    torch.cuda.synchronize()
    assert same((h, c), want) and same(got, seq)
