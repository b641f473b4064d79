"""The blocked Cholesky and triangular inverse of the orthonormalisations, at
the edges of their 16-column blocks, 32-row strips and waves."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _handle(J):
    from paper_1506_08147_amd import ALB
    return ALB([(12, 12, 12)], [(5.0, 5.0, 5.0)], [J], n_alb=[1])


def _gram(J, rng):
    Y = rng.standard_normal((4 * J, J)) * np.logspace(-2, 2, J)[None, :]
    return Y.T @ Y


@pytest.mark.parametrize("J", [1, 2, 15, 16, 17, 31, 32, 33, 48, 65, 127, 272, 511, 513, 544, 831, 832, 833])
def test_cholqr_orders(J):
    """T is upper triangular with a positive diagonal and T^T G T = I, to the
    backward error of a Cholesky factor of order J (condition ~9 after the
    diagonal scaling)."""
    import torch
    G = _gram(J, np.random.default_rng(J))
    h = _handle(J)
    T, fl = h.orthonormalise(0, torch.from_numpy(G).to("cuda:0"))
    T = T.cpu().numpy()
    h.close()
    assert list(fl[:4]) == [0, 0, 0, 0]
    assert np.all(np.tril(T, -1) == 0.0) and np.all(np.diag(T) > 0.0)
    assert np.abs(T.T @ G @ T - np.eye(J)).max() <= 1e-14 * (J + 10)


@pytest.mark.parametrize("J,p", [(17, 16), (40, 15), (40, 31), (50, 49)])
def test_cholqr_dependent_column(J, p):
    """A column p that repeats column 0 fails the pivot test of its block."""
    import torch
    G = _gram(J, np.random.default_rng(J))
    G[p, :] = G[0, :]
    G[:, p] = G[:, 0]
    G[p, p] = G[0, 0]
    h = _handle(J)
    _, fl = h.orthonormalise(0, torch.from_numpy(G).to("cuda:0"))
    _, fi = h.orthonormalise(0, torch.from_numpy(G).to("cuda:0"), init=True)
    h.close()
    assert fl[0] == 1 and fl[3] == 0
    assert fi[0] == 0 and fi[3] == 1
