"""GPU: steps of one batch entry in one launch (amq_cell1.hip) against the forms of two launches (results in place of the inputs,
operands already quantized), at the edges of chunks, slots and lanes, and with table rows that do not exist."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (64, 63), (65, 130), (130, 64), (256, 257), (300, 300), (512, 513), (650, 769), (1000, 1024), (1024, 1), (1025, 40),
          (40, 1025), (1100, 1537), (2048, 2048)]


@pytest.fixture(scope="module")
def amq():
    import paper_1802_00150_amd as m
    m.binding.lib()
    return m


def model(amq, gates, I, H, k_w):
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(I + 5 * H + gates)
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda:0")  # noqa: E731
    d = [*amq.quantize_weights(randn(gates * H, I) * 0.05, k_w, 2), *amq.quantize_weights(randn(gates * H, H) * 0.05, k_w, 2)]
    return d, [randn(gates * H) * 0.1 for _ in range(2)], randn(1, I), torch.tanh(randn(1, H)), randn(1, H)


@pytest.mark.parametrize("I,H", SHAPES)
def test_equal_to_two_launches(amq, I, H):
    import torch
    for k_w, k_a in ((2, 2), (3, 3), (2, 3), (3, 2)):
        for T in (2, 0):
            print("single step I=%d H=%d W%d/A%d T=%d" % (I, H, k_w, k_a, T), flush=True)
            d, b, x, h, c = model(amq, 4, I, H, k_w)
            h1, c1 = amq.lstm_step(*d, I, H, b[0], x, h, c, k_a, T)
            h2, c2 = h.clone(), c.clone()
            amq.lstm_step(*d, I, H, b[0], x, h2, c2, k_a, T, h_out=h2, c_out=c2)
            assert torch.equal(h1, h2) and torch.equal(c1, c2)
            d, b, x, h, _ = model(amq, 3, I, H, k_w)
            h1 = amq.gru_step(*d, I, H, *b, x, h, k_a, T)
            h2 = h.clone()
            amq.gru_step(*d, I, H, *b, x, h2, k_a, T, h_out=h2)
            assert torch.equal(h1, h2)
            assert torch.equal(amq.gru_step(*d, I, H, None, None, torch.zeros_like(x), torch.zeros_like(h), k_a, T),
                               torch.zeros_like(h))


@pytest.mark.parametrize("E,H,k", [(300, 200, 2), (1024, 1024, 3), (1030, 64, 2), (64, 2048, 3)])
def test_looked_up_input(amq, E, H, k):
    import torch
    vocab, V = 50, 97
    d, b, _, h, c = model(amq, 4, E, H, k)
    emb = amq.quantize_weights(torch.randn(vocab, E, device="cuda:0"), k, 2)
    soft = amq.quantize_weights(torch.randn(V, H, device="cuda:0") * 0.05, k, 2)
    for word in (0, vocab - 1, -1, vocab, 1 << 40):
        print("looked up E=%d H=%d k=%d word=%d" % (E, H, k, word), flush=True)
        ids = torch.tensor([word], device="cuda:0")
        hs, cs = h.clone(), c.clone()
        lp = amq.lm_step(*emb, E, *d, H, b[0], *soft, None, ids, hs, cs, k, k, 2)
        Xp, bx = amq.embedding_lookup(*emb, E, ids)
        if not 0 <= word < vocab:
            assert not Xp.any() and not bx.any()
        Hp, bh = amq.quantize_activations(h, k, 2)
        h2, c2 = amq.lstm_step_packed(*d, E, H, b[0], Xp, bx, Hp, bh, c)
        assert torch.equal(hs, h2) and torch.equal(cs, c2)
        want = torch.log_softmax(amq.binary_gemm(*soft, H, *amq.quantize_activations(h2, k, 2)).double(), dim=1)
        assert bool(((lp.double() - want).abs() <= 1e-5 * want.abs()).all())
