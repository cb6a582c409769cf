"""GPU: vectors whose pieces of 128 entries do not fill what the large kernels stage in LDS (amq_mfma32_body.h, amq_mfma4w.hip):
every number of pieces up to 8 with a full, a ragged and a one-entry last piece, columns and rows that fill no tile."""
import pytest

from test_gpu_large_steps import reference
from test_gpu_uneven_products import operands

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amq():
    import paper_1802_00150_amd as m
    m.binding.lib()
    return m


# 1 .. 8 pieces; one and two tiles of columns per wave, a wave with no row block, several per wave
@pytest.mark.parametrize("n", [100, 129, 256, 300, 385, 512, 513, 640, 700, 769, 896, 897, 1000, 1024])
@pytest.mark.parametrize("m,B,k_w,k_a", [(33000, 41, 2, 2), (9001, 130, 2, 3), (3001, 1000, 3, 3), (42000, 35, 3, 2)])
def test_products(amq, n, m, B, k_w, k_a):
    W, _, X, bias, ref = operands(amq, m, n, B, k_w, k_a)
    tol = 1e-4 * ref.abs() + 1e-4 * ref.pow(2).mean(1, keepdim=True).sqrt()
    Y = amq.binary_gemm(*W, n, *X, bias=bias)
    assert bool(((Y.double() - ref).abs() <= tol).all())


# amq_mfma32_body.h: three row blocks per SIMD, half of the SIMDs with five, one and two tiles of columns per wave
@pytest.mark.parametrize("n", [300, 650, 1000])
@pytest.mark.parametrize("m,B,k_w,k_a", [(10000, 256, 3, 2), (20000, 200, 2, 2), (20000, 200, 2, 3), (36000, 256, 2, 2)])
def test_precedence_by_row_blocks(amq, n, m, B, k_w, k_a):
    test_products(amq, n, m, B, k_w, k_a)


# amq_mfma4w.hip: eight, nine and twelve products per tile, at most four row blocks per wave and more
@pytest.mark.parametrize("n", [129, 1000])
@pytest.mark.parametrize("m,B", [(2000, 500), (9001, 70), (30001, 300)])
@pytest.mark.parametrize("k_w,k_a", [(2, 4), (3, 3), (3, 4), (4, 3), (4, 2)])
def test_many_products_per_tile(amq, n, m, B, k_w, k_a):
    test_products(amq, n, m, B, k_w, k_a)


# batches of the kernel with several tiles per wave: one, two and more row blocks per wave, units not a multiple of 4
@pytest.mark.parametrize("I,H,B,k_w,k_a", [(1, 1024, 256, 2, 2), (129, 1021, 250, 2, 2), (1024, 602, 600, 2, 2), (300, 1001, 200, 1, 3),
                                           (897, 1003, 161, 4, 1), (640, 1024, 190, 1, 1), (513, 1002, 130, 2, 4)])
def test_steps(amq, I, H, B, k_w, k_a):
    import torch
    for gates in (4, 3):
        print("staged step gates=%d I=%d H=%d B=%d W%d/A%d" % (gates, I, H, B, k_w, k_a), flush=True)
        g = torch.Generator(device="cuda:0").manual_seed(I + 3 * H + B)
        randn = lambda *s: torch.randn(*s, generator=g, device="cuda:0")  # noqa: E731
        d = [*amq.quantize_weights(randn(gates * H, I) * 0.04, k_w, 2), *amq.quantize_weights(randn(gates * H, H) * 0.04, k_w, 2)]
        bias = [randn(gates * H) * 0.1 for _ in range(2)]
        x, h, c = randn(B, I), torch.tanh(randn(B, H)), randn(B, H)
        h1, c1 = reference(amq, gates, I, H, d, bias, x, h, c, k_a)
        if gates == 4:
            got, gc = amq.lstm_step(*d, I, H, bias[0], x, h, c, k_a, 2)
            assert float((gc.double() - c1).abs().max()) < 1e-5
            amq.lstm_step(*d, I, H, bias[0], x, h, c, k_a, 2, h_out=h, c_out=c)  # in place
            assert torch.equal(h, got) and torch.equal(c, gc)
        else:
            got = amq.gru_step(*d, I, H, *bias, x, h, k_a, 2)
            amq.gru_step(*d, I, H, *bias, x, h, k_a, 2, h_out=h)
            assert torch.equal(h, got)
        # (hardware exponential and reciprocal: a few 1e-7 absolute; the exact integer sums add nothing)
        assert float((got.double() - h1).abs().max()) < 1e-5
