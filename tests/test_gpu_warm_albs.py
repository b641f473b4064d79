"""ALBs of the warm update with guard columns (a fixed number of iterations
from the vectors of the previous potential) against the oracle run the same
way, on starts for which W C_W, the direction after the first iteration, is
nearly rank deficient."""
import numpy as np
import pytest

import synth
from oracle import alb, lobpcg, teter
from oracle.hamiltonian import Operator

pytestmark = pytest.mark.gpu
GRID, WANTED, GUARD, NALB, EPS = (16, 16, 30), 56, 8, 20, 2.0 ** -52


def _filtered(op, J, seed):
    """Ritz vectors of three Chebyshev filters of degree 10 on a random block."""
    rng = np.random.default_rng(seed)
    n = int(np.prod(op.grid))
    x = np.random.default_rng(0).standard_normal((n, 1))
    for _ in range(60):
        x = op.apply(x)
        top = np.linalg.norm(x)
        x = x / top
    top *= 1.05 * 1.01
    X = np.linalg.qr(rng.standard_normal((n, J)))[0]
    for q in range(4):
        HX = op.apply(X)
        th, Q = np.linalg.eigh(X.T @ HX)
        X, HX = X @ Q, HX @ Q
        if q == 3:
            return X, top
        c, e = 0.5 * (top + th[-1]), 0.5 * (top - th[-1])
        s0 = s = e / (th[0] - c)
        Y0, Y1 = X, (HX - c * X) * (s / e)
        for _ in range(9):
            s2 = 1.0 / (2.0 / s0 - s)
            Y0, Y1, s = Y1, (op.apply(Y1) - c * Y1) * (2.0 * s2 / e) - (s * s2) * Y0, s2
        X = np.linalg.qr(Y1 / np.linalg.norm(Y1, axis=0))[0]


def _weakest(op, pre, X0):
    """Smallest eigenvalue of the second step's Schur complement of the first
    step's W against [X W]."""
    def direction(X):
        X = X @ lobpcg.scaled_cholqr(X)
        th, C = np.linalg.eigh(X.T @ op.apply(X))
        X = X @ C
        W = pre(op.apply(X) - X * th, X)
        W -= X @ (X.T @ W)
        return X, W @ lobpcg.scaled_cholqr(W)

    _, W1 = direction(X0)
    X, W2 = direction(lobpcg.lobpcg(op.apply, pre, X0, 1e-14, 1).X)
    Q = np.linalg.qr(np.hstack([X, W2]))[0]
    return np.linalg.svd(W1 - Q @ (Q.T @ W1), compute_uv=False)[-1] ** 2


@pytest.mark.parametrize("seed", [8, 11])
def test_warm_albs_match_oracle(seed):
    """Rounding of the Grams (EPS) grows by the reciprocal of the smallest
    eigenvalue of the P block's Schur complement (a factor 16 for its sums),
    and moves the wanted space by EPS ||H|| over its gap to the guard states;
    the ALBs follow the wanted space, within a factor 4 for their close
    singular values."""
    import torch
    from paper_1506_08147_amd import ALB
    dev = torch.device("cuda:0")
    J = WANTED + GUARD
    el = synth.single_element(seed=seed, grid=GRID, n_states=J, n_atoms=8)
    X0, top = _filtered(Operator(el.grid, el.box, el.V, el.kb), J, seed)
    V1 = synth.perturbed_potential(el, step=1)
    op = Operator(el.grid, el.box, V1, el.kb)
    pre = lambda R, X: teter.precondition(R, X, op.grid, op.box)  # noqa: E731
    ref = lobpcg.lobpcg(op.apply, pre, X0, 1e-14, 3, n_check=WANTED)
    bound = EPS * (16.0 / _weakest(op, pre, X0) + top / (ref.theta[WANTED] - ref.theta[WANTED - 1]))
    h = ALB([el.grid], [el.box], [J], tol=1e-6, max_iter=3, elem_lo=[el.elem_lo], elem_hi=[el.elem_hi],
            n_alb=[NALB], n_guard=GUARD)
    out = h.solve(torch.from_numpy(V1).to(dev), ALB.kb_batch([el.kb], dev),
                  torch.from_numpy(np.ascontiguousarray(X0.T)).reshape(-1).to(dev))
    st = out["stats"][0]
    assert st["iters"] == 3 and st["n_p_drop"] == 0
    X = out["eigvecs"].cpu().numpy().reshape(J, op.ng).T[:, :WANTED] * np.sqrt(op.dv)
    Xr = ref.X[:, :WANTED]
    off = np.linalg.norm(X - Xr @ (Xr.T @ X))
    A = out["albs"].cpu().numpy().reshape(NALB, -1).T
    Ar, sr = alb.restrict_svd(Xr, el.grid, el.elem_lo, el.elem_hi, op.dv, NALB)
    far = np.linalg.norm(A - Ar) / np.linalg.norm(Ar)
    print("wanted space off %.1e, ALBs %.1e, bound %.1e, singular values %.1e"
          % (off, far, bound, np.abs(out["sigma"].cpu().numpy() - sr).max()))
    assert off <= bound
    assert far <= 4.0 * bound
    assert np.abs(out["sigma"].cpu().numpy() - sr).max() <= bound
