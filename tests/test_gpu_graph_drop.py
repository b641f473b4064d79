"""Search directions dropped inside a captured graph: the products of the
iterations that follow run on a grid planned with them."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,seed", [((16, 16, 16), 0), ((16, 16, 16), 2), ((20, 20, 20), 2)])
def test_drop_inside_graph_equals_eager(grid, seed):
    """Projectors of two atoms on no local potential: the correction block
    loses rank before convergence.  The same 29 iterations, bit for bit."""
    import torch
    from paper_1506_08147_amd import ALB
    dev = torch.device("cuda:0")
    J = 16
    el = synth.single_element(seed=seed, grid=grid, n_states=J, n_atoms=2)
    X0 = torch.from_numpy(np.ascontiguousarray(el.X0.T)).reshape(-1).to(dev)
    V = torch.zeros(el.ng, dtype=torch.float64, device=dev)
    kbt = ALB.kb_batch([el.kb], dev)
    out = []
    for graph_iters in (0, 28):
        h = ALB([el.grid], [el.box], [J], tol=1e-14, max_iter=29, n_alb=[J // 2], graph_iters=graph_iters)
        out.append(h.solve(V, kbt, X0))
        h.close()
    se, sg = (o["stats"][0] for o in out)
    print("eager", se, "graph", sg)
    assert sg["graph_launches"] == 1 and sg["iters"] == se["iters"] == 29
    assert sg["n_p_drop"] == se["n_p_drop"] > 0
    assert sg["n_rr_fallback"] == se["n_rr_fallback"] and sg["max_res"] == se["max_res"]
    assert torch.equal(out[0]["eigvals"], out[1]["eigvals"]) and torch.equal(out[0]["eigvecs"], out[1]["eigvecs"])
