"""Orthonormalisation at the orders where the blocked factor takes over."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("J", [3, 7, 8, 9])
def test_cholqr_orders(J):
    """T^T G T = I to the backward error of a factor of order J; a repeated
    column fails the pivot test."""
    import torch
    from paper_1506_08147_amd import ALB
    Y = np.random.default_rng(J).standard_normal((4 * J, J)) * np.logspace(-2, 2, J)
    G = Y.T @ Y
    h = ALB([(12, 12, 12)], [(5.0, 5.0, 5.0)], [J], n_alb=[1])
    T, fl = h.orthonormalise(0, torch.from_numpy(G).to("cuda:0"))
    T = T.cpu().numpy()
    assert list(fl[:4]) == [0, 0, 0, 0] and np.all(np.tril(T, -1) == 0.0)
    assert np.abs(T.T @ G @ T - np.eye(J)).max() <= 1e-14 * (J + 10)
    Y[:, J - 1] = Y[:, 0]
    _, fl = h.orthonormalise(0, torch.from_numpy(Y.T @ Y).to("cuda:0"), init=True)
    assert fl[3] == 1
    h.close()
