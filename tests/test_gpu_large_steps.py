"""GPU: recurrent steps on 32 x 32 tiles (amq_mfma32_cell.hip) at the lines of their dispatch, with units and batches that fill no
tile, unequal blocks, blocks staged together and one after the other: every entry against binary64 products of the reconstructed
operands, and sequences of such steps against the step calls."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amq():
    import paper_1802_00150_amd as m
    m.binding.lib()
    return m


def reference(amq, gates, I, H, d, bias, x, h, c, k_a):
    """One step in binary64 on the GPU's own codes."""
    import torch

    def values(planes, alpha, n):
        bits = (planes.unsqueeze(-1) >> torch.arange(32, device=planes.device, dtype=torch.int32)) & 1
        signs = bits.reshape(*planes.shape[:2], -1)[:, :, :n].double() * 2 - 1
        return sum(signs[i] * alpha[:, i:i + 1].double() for i in range(planes.shape[0]))

    def product(v, planes, alpha, n):
        return values(*amq.quantize_activations(v, k_a, 2), n) @ values(planes, alpha, n).t().contiguous()

    gx, gh = product(x, d[0], d[1], I), product(h, d[2], d[3], H)
    if gates == 4:
        i, f, o, g = (gx + gh + bias[0].double()).split(H, dim=1)
        c1 = torch.sigmoid(f) * c.double() + torch.sigmoid(i) * torch.tanh(g)
        return torch.sigmoid(o) * torch.tanh(c1), c1
    xr, xz, xn = (gx + bias[0].double()).split(H, dim=1)
    hr, hz, hn = (gh + bias[1].double()).split(H, dim=1)
    z = torch.sigmoid(xz + hz)
    n = torch.tanh(xn + torch.sigmoid(xr + hr) * hn)
    return (1 - z) * n + z * h.double(), None


# (I, H, B): one wave more and fewer than the lines, H % 8 and % 4, B % 32, blocks of 300 and 2000 entries, LDS shared
SHAPES = [(1024, 1024, 256, 2, 3), (1024, 1024, 193, 2, 3), (700, 1021, 257, 2, 3), (650, 650, 250, 3, 3), (1024, 1030, 225, 3, 3),
          (1100, 1100, 250, 2, 2), (2048, 2048, 256, 2, 2), (2048, 2047, 129, 3, 3), (300, 2000, 128, 3, 3), (2000, 333, 520, 2, 3),
          (1300, 1306, 127, 2, 2), (1500, 1500, 225, 3, 2), (1025, 64, 2600, 2, 2), (1, 1500, 200, 2, 2),
          # workgroups of four waves beyond one for every compute unit; a second round nearly empty and nearly full; a third
          (900, 900, 272, 3, 3), (900, 900, 140, 3, 3), (2048, 2048, 272, 3, 2), (2048, 2048, 400, 2, 3), (1024, 1024, 600, 2, 3),
          (1024, 1024, 1000, 3, 3), (2048, 2000, 560, 2, 2)]


@pytest.mark.parametrize("I,H,B,k_w,k_a", SHAPES)
def test_steps(amq, I, H, B, k_w, k_a):
    import torch
    for gates in (4, 3):
        print("large step gates=%d I=%d H=%d B=%d W%d/A%d" % (gates, I, H, B, k_w, k_a), flush=True)
        g = torch.Generator(device="cuda:0").manual_seed(I + 3 * H + B)
        randn = lambda *s: torch.randn(*s, generator=g, device="cuda:0")  # noqa: E731
        d = [*amq.quantize_weights(randn(gates * H, I) * 0.04, k_w, 2), *amq.quantize_weights(randn(gates * H, H) * 0.04, k_w, 2)]
        bias = [randn(gates * H) * 0.1 for _ in range(2)]
        x, h, c = randn(B, I), torch.tanh(randn(B, H)), randn(B, H)
        h1, c1 = reference(amq, gates, I, H, d, bias, x, h, c, k_a)
        if gates == 4:
            got, gc = amq.lstm_step(*d, I, H, bias[0], x, h, c, k_a, 2)
            assert float((gc.double() - c1).abs().max()) < 1e-5
            hs, hp, cp = torch.empty((2, B, H), device=h.device), h.clone(), c.clone()
            xs = torch.stack([x, x.flip(0)])
            amq.lstm_sequence(*d, I, H, bias[0], xs, hp, cp, k_a, 2, hs=hs)
            h2, c2 = amq.lstm_step(*d, I, H, bias[0], xs[1].contiguous(), got, gc, k_a, 2)
            assert torch.equal(hs[0], got) and torch.equal(hs[1], h2) and torch.equal(hp, h2) and torch.equal(cp, c2)
        else:
            got = amq.gru_step(*d, I, H, *bias, x, h, k_a, 2)
            hs, hp = torch.empty((2, B, H), device=h.device), h.clone()
            xs = torch.stack([x, x.flip(0)])
            amq.gru_sequence(*d, I, H, *bias, xs, hp, k_a, 2, hs=hs)
            h2 = amq.gru_step(*d, I, H, *bias, xs[1].contiguous(), got, k_a, 2)
            assert torch.equal(hs[0], got) and torch.equal(hs[1], h2) and torch.equal(hp, h2)
        # (hardware exponential and reciprocal: a few 1e-7 absolute; sums of at most 9 products with 24-bit factors below that)
        assert float((got.double() - h1).abs().max()) < 1e-5


@pytest.mark.parametrize("gates,I,H,B,k_w,k_a", [(4, 1100, 1100, 250, 2, 2), (3, 1024, 1024, 256, 2, 3)])
def test_state_at_any_float(amq, gates, I, H, B, k_w, k_a):
    """The tensors of the state may begin at any multiple of four bytes, each for itself."""
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(I + B)
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda:0")  # noqa: E731
    d = [*amq.quantize_weights(randn(gates * H, I) * 0.04, k_w, 2), *amq.quantize_weights(randn(gates * H, H) * 0.04, k_w, 2)]
    x, h, c = randn(B, I), torch.tanh(randn(B, H)), randn(B, H)

    def place(offset, values=None):
        room = torch.full((B * H + 8,), 7.0, device="cuda:0")
        t = room[offset:offset + B * H].view(B, H)
        return room, t if values is None else t.copy_(values)

    def step(h_at, c_at, ho_at, co_at):
        rooms = [place(ho_at), place(co_at)]
        if gates == 4:
            amq.lstm_step(*d, I, H, None, x, place(h_at, h)[1], place(c_at, c)[1], k_a, 2, h_out=rooms[0][1], c_out=rooms[1][1])
        else:
            amq.gru_step(*d, I, H, None, None, x, place(h_at, h)[1], k_a, 2, h_out=rooms[0][1])
        for (room, _), at in zip(rooms, (ho_at, co_at)):  # nothing around them is written
            assert bool((room[:at] == 7.0).all()) and bool((room[at + B * H:] == 7.0).all())
        return [t for _, t in rooms[:2 if gates == 4 else 1]]

    want = step(0, 0, 0, 0)
    for at in ((1, 0, 0, 0), (0, 3, 0, 0), (0, 0, 2, 0), (0, 0, 0, 1), (3, 1, 2, 3)):
        print("state at", at, flush=True)
        assert all(torch.equal(a, b) for a, b in zip(step(*at), want))
