"""Density and nonlocal block of arbitrary columns at the edges of their tiles:
16-column and 16-row blocks of the density product, boxes at the start, the end
and all of the grid for the scatter."""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import dgblocks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 65, 130])
@pytest.mark.parametrize("grid,lo,hi", [((8, 6, 10), (0, 0, 0), (8, 6, 10)), ((10, 9, 6), (3, 2, 0), (8, 9, 5)),
                                        ((36, 30, 20), (0, 11, 7), (1, 30, 8)), ((20, 36, 18), (7, 1, 2), (20, 35, 16))])
def test_density_and_nonlocal_tiles(grid, lo, hi, n):
    import torch
    from paper_1506_08147_amd import ALB
    ne = int(np.prod(np.subtract(hi, lo)))
    if n > ne:
        pytest.skip("more columns than rows")
    dev = torch.device("cuda:0")
    e = synth.single_element(seed=7, grid=grid, n_states=n, n_atoms=3)
    h = ALB([grid], [e.box], [n], elem_lo=[lo], elem_hi=[hi], n_alb=[n])
    h.set_potential(torch.from_numpy(e.V).to(dev), ALB.kb_batch([e.kb], dev))
    rng = np.random.default_rng(n)
    phi, P = rng.standard_normal((ne, n)), rng.standard_normal((n, n))
    dphi = torch.from_numpy(np.ascontiguousarray(phi.T).ravel()).to(dev)
    rho = h.density(dphi, torch.from_numpy(np.ascontiguousarray(P.T).ravel()).to(dev)).cpu().numpy()
    # two sums of n products each, in any order
    bound = 2.0 * (2 * n + 4) * 2.0 ** -53 * np.einsum("ri,ij,rj->r", np.abs(phi), np.abs(P), np.abs(phi))
    assert np.all(np.abs(rho - dgblocks.density(phi, P)) <= bound)
    H = h.nonlocal_block(dphi).cpu().numpy().reshape(n, n, order="F")
    ref = dgblocks.nonlocal_block(phi, e.kb, grid, lo, hi, e.dv)
    # projections are sums over at most all grid points
    size = dgblocks.nonlocal_block(np.abs(phi), _absolute(e.kb), grid, lo, hi, e.dv)
    assert np.all(np.abs(H - ref) <= 4.0 * (int(np.prod(grid)) + 100) * 2.0 ** -53 * size + 1e-300)
    h.close()


def _absolute(kb):
    return dataclasses.replace(kb, val=np.abs(kb.val), gamma=np.abs(kb.gamma))
