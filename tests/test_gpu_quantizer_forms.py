"""GPU: the quantizer's two forms, one for few vectors and one for many, to the bit alike on both sides of the line between them,
and alike when the same vectors arrive in calls of other counts."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_coef_close, compare_codes, host, planes_host, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 3, 4])
@pytest.mark.parametrize("n", [1, 64, 65, 128, 129, 511, 513, 896, 897, 1023, 1024, 1025, 2047, 2048, 2049, 2176, 3001, 3584, 3585, 4095, 4096])
def test_few_and_many_vectors_alike(k, n):
    import torch

    import paper_1802_00150_amd as amq
    g = np.random.default_rng(97 * n + k)
    X = to_dev(np.tanh(g.standard_normal((768, n))).astype(np.float32))
    for T in (2, 0):
        P, A = amq.quantize_activations(X, k, T)
        R = amq.fake_quantize(X, k, T)
        first = host(X[:5])
        pr, ar = oracle.quantize_rows(first, k, T)
        assert_coef_close(host(A[:5]), ar)
        compare_codes(first, planes_host(P[:, :5].contiguous()), pr, ar)
        for rows in (1, 3, 256, 257, 599, 600, 767):  # the line: 600 vectors, 768 at k = 3 and some lengths, 256 beyond 2048
            print("forms k=%d n=%d T=%d rows=%d" % (k, n, T, rows), flush=True)
            p, a = amq.quantize_activations(X[:rows].contiguous(), k, T)
            assert torch.equal(p, P[:, :rows]) and torch.equal(a, A[:rows])
            assert torch.equal(amq.fake_quantize(X[:rows].contiguous(), k, T), R[:rows])
