"""The operator at the edges of its projector handling: column counts around
the blocks of four, one atom and more projectors than the epilogue keeps in LDS
(256), grids of fewer and more points than a workgroup's lanes."""
import numpy as np
import pytest

import synth
from oracle.hamiltonian import Operator

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cols", [1, 3, 4, 5, 8])
@pytest.mark.parametrize("grid,atoms", [((6, 8, 5), 1), ((12, 10, 9), 80), ((36, 32, 8), 3), ((48, 40, 6), 80),
                                        ((60, 48, 4), 80)])
def test_operator_projectors(grid, atoms, cols):
    import torch
    from paper_1506_08147_amd import ALB
    dev = torch.device("cuda:0")
    e = synth.single_element(seed=3, grid=grid, n_states=cols, n_atoms=atoms)
    h = ALB([grid], [e.box], [cols], n_alb=[1])
    h.set_potential(torch.from_numpy(e.V).to(dev), ALB.kb_batch([e.kb], dev))
    X = np.random.default_rng(cols).standard_normal((int(np.prod(grid)), cols))
    HX = h.apply_h(0, torch.from_numpy(np.ascontiguousarray(X.T)).to(dev)).cpu().numpy().T
    ref = Operator(e.grid, e.box, e.V, e.kb).apply(X)
    assert np.abs(HX - ref).max() < 1e-13 * np.abs(ref).max()
    h.close()
