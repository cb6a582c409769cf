"""GPU: the output layer of one batch entry at every number of row groups per wave (amq_bmv_online.hip), on either side of the lines
between them, with rows that fill no group and workgroups with waves that have none; plain products on either side of theirs
(amq_bmv.hip)."""
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


# 2047 quarters of the waves, 2048, a row and a half group more; one vector, few and the most that this kernel takes
@pytest.mark.parametrize("m,n", [(2 * 8188, 4096), (2 * 8188 + 1, 4000), (2 * 8192 + 5, 2100), (4 * 8188, 2048), (4 * 8188 + 1, 1025),
                                 (4 * 8188 + 7, 1999), (8 * 8188 + 3, 1024), (16385, 8192)])
@pytest.mark.parametrize("B,k_w,k_a", [(1, 2, 2), (1, 3, 3), (2, 2, 3), (4, 1, 4), (16, 3, 2), (1, 4, 4), (1, 4, 1), (2, 2, 1)])
def test_products(amq, m, n, B, k_w, k_a):
    import torch
    W, _, X, bias, ref = operands(amq, m, n, B, k_w, k_a)
    tol = 1e-4 * ref.abs() + 1e-4 * ref.pow(2).mean(1, keepdim=True).sqrt()
    Y = amq.binary_gemm(*W, n, *X, bias=bias)
    assert bool(((Y.double() - ref).abs() <= tol).all())
    # half of the rows at a time are fewer waves than the line, and the same sums
    h = m // 2
    parts = [amq.binary_gemm(W[0][:, r].contiguous(), W[1][r].contiguous(), n, *X, bias=bias[r]) for r in (slice(0, h), slice(h, m))]
    if n > 1024 or B <= 4:  # (else the matrix cores)
        assert torch.equal(torch.cat(parts, 1), Y)
