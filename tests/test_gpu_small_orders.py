"""The smallest orders of the eigensolver, in one launch, and eigenvalue counts
around the eight of a bisection workgroup and the sixteen columns of a
back-transformation workgroup."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(1, 1), (2, 2), (3, 1), (4, 4), (5, 1), (5, 5), (6, 3), (200, 7), (200, 8), (200, 9),
                                 (200, 15), (200, 16), (200, 17), (520, 8), (520, 9)])
def test_syev_orders(n, k):
    """Backward error and orthogonality in units of rounding times the order."""
    import torch
    from paper_1506_08147_amd import small_syev
    M = np.random.default_rng(n + 31 * k).standard_normal((5, n, n))
    M = M + M.transpose(0, 2, 1)
    w, Z = small_syev(torch.from_numpy(M).to("cuda:0"), k)
    w, Z = w.cpu().numpy(), Z.cpu().numpy()
    for i in range(5):
        ref = np.linalg.eigvalsh(M[i])
        sc = max(1.0, np.abs(ref).max())
        Zi = Z[i].T
        assert np.abs(w[i][:k] - ref[:k]).max() <= 1e-13 * sc * n
        assert np.abs(M[i] @ Zi - Zi * w[i][:k]).max() <= 1e-12 * sc * np.sqrt(n)
        assert np.abs(Zi.T @ Zi - np.eye(k)).max() <= 1e-12 * np.sqrt(n)
