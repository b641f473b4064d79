"""The operator's projector epilogue over the sizes of groups that share a
support (its entries are stored as wide as the largest), on planes of each FFT
tile, and without projectors."""
import numpy as np
import pytest

import synth
from oracle.hamiltonian import Operator

pytestmark = pytest.mark.gpu


def _kb(grid, box, sizes, rng):
    """Groups of the given sizes on random supports, one of them empty."""
    ng = int(np.prod(grid))
    dv = float(np.prod(box)) / ng
    ptr, idx, val = [0], [], []
    for g, size in enumerate(sizes):
        sup = np.sort(rng.choice(ng, 0 if g == 1 else rng.integers(1, ng // 2), replace=False)).astype(np.int32)
        for _ in range(size):
            b = rng.standard_normal(sup.size)
            idx.append(sup)
            val.append(b / np.sqrt(dv * max(b @ b, 1e-300)))
            ptr.append(ptr[-1] + sup.size)
    return synth.KB(gamma=rng.uniform(-1.0, 1.0, len(ptr) - 1), ptr=np.asarray(ptr, np.int64),
                    idx=np.concatenate(idx), val=np.concatenate(val))


@pytest.mark.parametrize("sizes", [(), (1, 1, 1), (2, 1, 2), (3, 4), (5, 2, 1), (8, 3, 8), (9, 1)])
@pytest.mark.parametrize("grid", [(6, 8, 5), (36, 32, 4), (48, 48, 4), (60, 48, 4)])
def test_operator_group_sizes(grid, sizes):
    import torch
    from paper_1506_08147_amd import ALB
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(len(sizes) + sum(sizes))
    box = tuple(0.6 * n for n in grid)
    kb = _kb(grid, box, sizes, rng) if sizes else synth.KB(np.zeros(0), np.zeros(1, np.int64), np.zeros(0, np.int32),
                                                            np.zeros(0))
    V = rng.standard_normal(int(np.prod(grid)))
    X = rng.standard_normal((V.size, 5))
    ref = Operator(grid, box, V, kb).apply(X)
    for precision, tol in (("fp64", 1e-13), ("mixed", 1e-5)):
        h = ALB([grid], [box], [5], n_alb=[1], precision=precision)
        h.set_potential(torch.from_numpy(V).to(dev), ALB.kb_batch([kb], dev) if sizes else None)
        HX = h.apply_h(0, torch.from_numpy(np.ascontiguousarray(X.T)).to(dev)).cpu().numpy().T
        assert np.abs(HX - ref).max() < tol * np.abs(ref).max()
        h.close()
