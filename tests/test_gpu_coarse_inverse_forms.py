"""The coarsest inverse's register form, 145 to 288 free DOFs: its smallest
size, sizes with no tile beside the diagonal in LDS, exactly as many off-diagonal
tiles as the registers hold (120, at 252 DOFs), some in LDS, the largest, and
the first size of the form in memory.  Against the oracle's direct solution;
tolerance: both are unpivoted eliminations of the same SPD system in FP64,
each within n eps kappa of the exact solution."""
import numpy as np
import pytest
import torch

from oracle import ke as oke, mesh, operator as op
from paper_2607_26382_amd import topoguard as tg

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("floor", [1e-3, 1e-6])
@pytest.mark.parametrize("dims", [(3, 4, 3), (13, 1, 1), (17, 1, 1), (21, 1, 1), (22, 1, 1), (23, 1, 1), (24, 1, 1),
                                  (5, 3, 3), (25, 1, 1)])
def test_inverse_equals_direct_solution(dims, floor):
    rng = np.random.default_rng(4)
    og = mesh.Grid(*dims)
    rho = np.where(rng.random(og.n_elem) < 0.3, 0.0, rng.random(og.n_elem))
    free = og.free_dofs()
    n = int(free.sum())
    assert 144 < n <= 300
    K = op.free_block(op.assemble(og, op.young(rho, 3.0, floor), oke.ke()), free)
    r = np.where(free, rng.standard_normal(og.n_dof), 0.0)
    g = tg.Grid(*dims, max_restart=1, device=DEV)
    assert g.n_levels == 1
    g.set_density(torch.tensor(rho, device=DEV), 3.0, floor)
    x = op.solve_direct(K, r[free])
    kappa = np.linalg.cond(K.toarray())
    z = g.vcycle(torch.tensor(r, device=DEV)).cpu().numpy()
    err = np.linalg.norm(z[free] - x) / np.linalg.norm(x)
    print(dims, n, floor, f"err {err:.2e} bound {2 * n * np.finfo(float).eps * kappa:.2e}", flush=True)
    assert np.all(z[~free] == 0.0)
    assert err <= 2 * n * np.finfo(float).eps * kappa
