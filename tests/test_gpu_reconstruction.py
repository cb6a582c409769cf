"""GPU: the reconstruction that the quantizer reads off its code table by position equals what the codes and coefficients of the
same rows give, bit for bit -- also where Gram matrices are singular, coefficients negative or equal, and orders unusual."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 3, 4])
@pytest.mark.parametrize("n", [3, 64, 128, 300, 513, 650, 1024, 1025, 2048, 4100])
def test_equal_to_codes_and_coefficients(k, n):
    import torch

    import paper_1802_00150_amd as amq
    print("reconstruction k=%d n=%d" % (k, n), flush=True)
    g = np.random.default_rng(17 * n + k)
    base = g.standard_normal((9, n)).astype(np.float32)
    base[1] = -0.25                                          # constant: planes coincide
    base[2] = np.where(np.arange(n) % 3 == 0, -0.0, 0.0)     # zeros of both signs
    base[3] = g.integers(-3, 4, n)                           # values that meet midpoints exactly
    base[4, 0] = 1e4                                         # one entry dominates: unusual order of the code table
    base[5] = np.abs(base[5])
    base[6] = base[6] ** 3
    base[7] = np.where(np.arange(n) % 2 == 0, 0.25, -0.25)
    base[8] = np.sign(base[8]) * (1 + (np.arange(n) % 2))    # two magnitudes: two planes are exact, the others singular
    for rows in (9, 1035):                                   # the latency form and the throughput form
        W = to_dev(np.ascontiguousarray(np.tile(base, (rows // 9, 1))))
        for T in (0, 1, 2, 3):
            assert torch.equal(amq.fake_quantize(W, k, T), amq.dequantize(*amq.quantize_weights(W, k, T), n)), (rows, T)
