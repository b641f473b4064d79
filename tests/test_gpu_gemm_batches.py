"""Batches of block products whose partial sums are shared by several launches,
and coefficient matrices past the reach of 32-bit byte offsets."""
import pytest

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


def test_gram_batch_in_launches_equals_single():
    """130 products of 17 chunks of 96 x 32: two launches of 65; each product
    bit for bit that of a batch of one."""
    import torch
    from paper_1506_08147_amd import gemm_batched
    g = torch.Generator(device="cuda:0").manual_seed(5)
    A = torch.randn(130, 96, 13824, dtype=torch.float64, device="cuda:0", generator=g)
    B = torch.randn(130, 32, 13824, dtype=torch.float64, device="cuda:0", generator=g)
    C = gemm_batched(1, A, B)
    for i in (0, 1, 64, 65, 66, 129):
        assert torch.equal(C[i], gemm_batched(1, A[i:i + 1].contiguous(), B[i:i + 1].contiguous())[0])
        bound = (13824 + 2) * EPS * (B[i].abs() @ A[i].abs().t().contiguous())
        assert bool(((C[i] - B[i] @ A[i].t().contiguous()).abs() <= 2.0 * bound).all())


def test_update_of_many_rows_of_coefficients():
    """Y = A C with 2^22 rows of C: the last columns of a 144-column tile lie
    more than 4 GiB from its first."""
    import torch
    from paper_1506_08147_amd import gemm_batched
    m, n, K = 1 << 22, 144, 16
    g = torch.Generator(device="cuda:0").manual_seed(6)
    A = torch.randn(1, m, K, dtype=torch.float64, device="cuda:0", generator=g)
    C = torch.randn(1, n, m, dtype=torch.float64, device="cuda:0", generator=g)
    Y = gemm_batched(0, A, C)[0]
    for j in (0, 15, 16, 127, 128, 129, 143):
        # each row's sum of m products in any order
        ref, mag = (A[0] * C[0, j, :, None]).sum(0), (A[0] * C[0, j, :, None]).abs().sum(0)
        assert bool(((Y[j] - ref).abs() <= 2.0 * (m + 2) * EPS * mag).all()), j
