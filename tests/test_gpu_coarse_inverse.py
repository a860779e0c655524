"""The coarsest level's explicit inverse at the sizes where its form or its
tiling changes: below one 16 x 16 tile, partly filled last tiles, a whole
number of tiles, the largest size held in LDS (144), sizes beyond it and the
largest direct one (510 of 512).  A one-level grid's V-cycle is that inverse,
so z = V(r) is compared with the oracle's direct solution of the assembled
matrix.  Tolerance: both are solutions of the same SPD system by unpivoted
elimination in FP64, each within n eps kappa of the exact one."""
import numpy as np
import pytest
import torch

from oracle import ke as oke, mesh, operator as op
from paper_2607_26382_amd import topoguard as tg

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _case(dims, floor, seed):
    rng = np.random.default_rng(seed)
    og = mesh.Grid(*dims)
    rho = np.where(rng.random(og.n_elem) < 0.3, 0.0, rng.random(og.n_elem))
    free = og.free_dofs()
    K = op.free_block(op.assemble(og, op.young(rho, 3.0, floor), oke.ke()), free)
    r = np.where(free, rng.standard_normal(og.n_dof), 0.0)
    return rho, free, K, r


@pytest.mark.parametrize("floor", [1e-3, 1e-6])
@pytest.mark.parametrize("dims", [(1, 1, 1), (2, 1, 1), (2, 2, 2), (4, 2, 2), (4, 3, 2), (3, 3, 3), (5, 3, 2),
                                  (6, 3, 3), (7, 4, 3), (17, 1, 4)])
def test_inverse_equals_direct_solution(dims, floor):
    rho, free, K, r = _case(dims, floor, 11)
    g = tg.Grid(*dims, max_restart=1, device=DEV)
    assert g.n_levels == 1 and g.info.coarse_free_dof == free.sum()
    g.set_density(torch.tensor(rho, device=DEV), 3.0, floor)
    z = g.vcycle(torch.tensor(r, device=DEV)).cpu().numpy()
    x = op.solve_direct(K, r[free])
    n = free.sum()
    kappa = np.linalg.cond(K.toarray())
    err = np.linalg.norm(z[free] - x) / np.linalg.norm(x)
    print(dims, n, floor, f"err {err:.2e} bound {2 * n * np.finfo(float).eps * kappa:.2e}", flush=True)
    assert np.all(z[~free] == 0.0)
    assert err <= 2 * n * np.finfo(float).eps * kappa


def test_batched_inverse_is_bitwise_the_single_one():
    dims = [(6, 3, 3), (4, 2, 2), (17, 1, 4), (4, 3, 2)]
    grids, rhos, single = [], [], []
    for i, d in enumerate(dims):
        rho, _, _, r = _case(d, 1e-3, 20 + i)
        g = tg.Grid(*d, max_restart=1, device=DEV)
        g.set_density(torch.tensor(rho, device=DEV), 3.0, 1e-3)
        single.append((torch.tensor(r, device=DEV), g.vcycle(torch.tensor(r, device=DEV))))
        rhos.append(torch.tensor(rho, device=DEV))
        grids.append(g)
    b = tg.Batch(grids)
    b.set_density(rhos, 3.0, [1e-3] * len(dims))
    for g, (r, z) in zip(grids, single):
        assert torch.equal(g.vcycle(r), z)
