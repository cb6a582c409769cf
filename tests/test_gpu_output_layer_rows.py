"""GPU: the output layer of one batch entry at every number of row groups per wave (amq_bmv_online.hip), on either side of the lines
between them, with rows that fill no group and workgroups with waves that have none."""
import pytest

from test_gpu_uneven_products import operands

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amq():
    import paper_1802_00150_amd as m
    m.binding.lib()
    return m


# row groups of 4 (1025 to 2048 entries), 8 and 64 rows: up to 1024, 2048, 3072, 4096, 6144, 8192, 12288 of them and one more
@pytest.mark.parametrize("V,n", [(8192, 1024), (8193, 600), (4 * 2048, 2048), (4 * 2048 + 1, 1025), (8 * 3072, 1000), (8 * 3072 + 1, 1024),
                                 (8 * 4096, 513), (8 * 4096 + 3, 640), (4 * 6144, 2000), (4 * 6144 + 1, 2048), (4 * 8192, 1100),
                                 (4 * 8192 + 2, 2048), (4 * 12288, 1030), (4 * 12288 + 1, 1030), (64 * 1024 + 5, 100)])
@pytest.mark.parametrize("k_w,k_a", [(2, 2), (2, 3), (3, 2), (3, 3)])
def test_log_probabilities(amq, V, n, k_w, k_a):
    import torch
    W, x, _, bias, ref = operands(amq, V, n, 1, k_w, k_a)
    want = torch.log_softmax(ref, 1)
    got = amq.softmax_layer(*W, n, bias, x, k_a, 2)
    # (logits: binary32 sums of 128-entry chunks; exponentials and logarithm a few 1e-6 absolute)
    tol = 1e-4 * ref.pow(2).mean().sqrt() + 1e-5 * want.abs()
    assert bool(((got.double() - want).abs() <= tol).all())
    assert torch.equal(amq.softmax_layer(*W, n, bias, x, k_a, 2), got)
