"""Block products with coefficient matrices past the reach of 32-bit byte offsets."""
import pytest

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


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
