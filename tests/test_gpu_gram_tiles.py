"""The block products A^T B at the edges of their tiles: row blocks and tiles
of 64 and 128, column blocks of 16, stages of 16 rows and split chunks, with
columns at 16-byte boundaries (even K) and not (odd K)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 2, 15, 16, 17, 31, 32, 33, 48, 250, 2167, 2168, 4336, 4337, 13824, 13825])
@pytest.mark.parametrize("m,n", [(1, 1), (16, 17), (17, 16), (64, 31), (65, 144), (113, 145), (128, 96), (129, 128),
                                 (145, 80), (272, 272)])
def test_gram_tiles(K, m, n):
    import torch
    from paper_1506_08147_amd import gemm_batched
    rng = np.random.default_rng(K + 7 * m + 31 * n)
    A, B = rng.standard_normal((2, m, K)), rng.standard_normal((2, n, K))
    C = gemm_batched(1, torch.from_numpy(A).to("cuda:0"), torch.from_numpy(B).to("cuda:0")).cpu().numpy()
    for i in range(2):
        # backward error of a sum of K products, in any order
        bound = (K + 2) * 2.0 ** -53 * (np.abs(B[i]) @ np.abs(A[i]).T) + 1e-300
        assert np.all(np.abs(C[i] - B[i] @ A[i].T) <= 2.0 * bound)


@pytest.mark.parametrize("K", [1, 2, 127, 128, 129, 130, 256, 1000, 1001])
@pytest.mark.parametrize("m,n", [(1, 1), (2, 16), (15, 17), (16, 31), (17, 144), (33, 145), (48, 96), (81, 128),
                                 (272, 272)])
def test_update_tiles(K, m, n):
    """Y = alpha A C + beta Y at the edges of the 128-row tiles, 16-column
    blocks and 16-deep stages, for even and odd leading dimensions."""
    import torch
    from paper_1506_08147_amd import gemm_batched
    rng = np.random.default_rng(K + 7 * m + 31 * n)
    A, B = rng.standard_normal((2, m, K)), rng.standard_normal((2, n, m))
    Y0 = rng.standard_normal((2, n, K))
    dev = "cuda:0"
    for alpha, beta in ((1.0, 0.0), (-0.7, 1.3)):
        Y = gemm_batched(0, torch.from_numpy(A).to(dev), torch.from_numpy(B).to(dev), alpha=alpha, beta=beta,
                         Cin=torch.from_numpy(Y0).to(dev)).cpu().numpy()
        for i in range(2):
            ref = alpha * (B[i] @ A[i]) + beta * Y0[i]
            bound = (m + 4) * 2.0 ** -53 * (abs(alpha) * (np.abs(B[i]) @ np.abs(A[i])) + abs(beta * Y0[i]))
            assert np.all(np.abs(Y[i] - ref) <= 2.0 * bound)
