"""GPU: the quantizer's wide register forms (20 to 32 slots per lane, one wave or two per vector), at the edges of slots and forms and
of the numbers of vectors from which they are used, against the oracle; and the reconstruction against codes and coefficients."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_coef_close, compare_codes, host, planes_host, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [2, 3, 4])
@pytest.mark.parametrize("rows", [1535, 1536, 1537, 2048, 2049, 2700, 4096, 12288])
def test_wide_forms_and_special_rows(k, rows):
    import torch

    import paper_1802_00150_amd as amq
    many = (1025, 1152, 1153, 1280, 1281, 1500, 1536, 1537, 1792, 1793, 2000, 2048, 2049, 2304, 2560, 2561, 3000, 3072)
    lengths = {1535: (1100, 3000), 1536: many, 1537: many if k == 4 else (1100,), 2048: (1700, 2048), 2049: (1700, 2048),
               2700: (1700, 2048), 4096: (2561, 3072, 3073, 3333, 3584, 3585, 4000, 4096), 12288: (3100, 4096)}[rows]
    for n in lengths:
        print("wide k=%d rows=%d n=%d" % (k, rows, n), flush=True)
        g = np.random.default_rng(31 * n + k)
        base = g.standard_normal((8, n)).astype(np.float32)
        base[1] = -0.25                                          # constant: every further residual is exactly zero
        base[2] = np.where(np.arange(n) % 3 == 0, -0.0, 0.0)     # zeros of both signs
        base[3] = g.integers(-3, 4, n)                           # values that can meet a midpoint exactly
        base[4, 0] = 1e4                                         # one entry dominates: unusual order of the code table
        base[5] = np.abs(base[5])                                # one-sided
        base[6] = base[6] ** 3                                   # heavy tails
        base[7] = np.where(np.arange(n) % 2 == 0, 0.25, -0.25)   # planes coincide
        W = to_dev(base).repeat(rows // 8, 1)
        W = torch.cat([W, W[:rows - W.shape[0]]]).contiguous()
        for T in (2, 0):
            pr, ar = oracle.quantize_rows(base, k, T)
            pg, ag = amq.quantize_weights(W, k, T)
            for r in range(8):                                   # equal rows give equal results
                assert bool((pg[:, r::8] == pg[:, r:r + 1]).all()) and bool((ag[r::8] == ag[r]).all())
            assert_coef_close(host(ag[:8]), ar)
            compare_codes(base, planes_host(pg[:, :8].contiguous()), pr, ar)
            assert torch.equal(amq.fake_quantize(W, k, T), amq.dequantize(pg, ag, n))
