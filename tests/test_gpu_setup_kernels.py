"""The set-up's kernels where their split changes: a workgroup takes one element
of a Galerkin level, or eight from 16384 elements on (64x64x32 has just that
many at level 1, 54x54x54 a number that eight does not divide, at a level that
cannot be coarsened on), the node blocks and mode-basis elements of every level
and of a batch's problems share one launch.  What the matrices give is compared
with the oracle: the FP64 cycle to 1e-9 of its largest entry as elsewhere, and a
problem's set-up in a batch with the same problem alone, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import ke as oke, mesh, multigrid as omg, operator as op
from paper_2607_26382_amd import topoguard as tg
from paper_2607_26382_amd._lib import TopoguardError

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dims", [(4, 2, 2), (8, 4, 4), (24, 12, 12), (8, 16, 4), (40, 16, 24), (64, 64, 32)])
def test_cycle_of_new_setup(dims):
    print(f"setup {dims}", flush=True)
    rng = np.random.default_rng(2)
    og = mesh.Grid(*dims)
    rho, free = rng.random(og.n_elem), og.free_dofs()
    g = tg.Grid(*dims, max_restart=1, device=DEV)
    g.set_density(torch.tensor(rng.random(og.n_elem), device=DEV), 3.0, 1e-2)   # replaced below
    g.set_density(torch.tensor(rho, device=DEV), 3.0, 1e-3)
    H = omg.build_hierarchy(og, op.young(rho, 3.0, 1e-3), oke.ke())
    r = np.zeros(og.n_dof)
    r[free] = rng.standard_normal(int(free.sum()))
    ref = omg.vcycle(H, r[free])
    z = g.vcycle(torch.tensor(r, device=DEV), tg.F64).cpu().numpy()
    assert np.abs(z[free] - ref).max() <= 1e-9 * np.abs(ref).max()


def test_remainder_of_a_level_without_cycle():
    print("setup 54x54x54", flush=True)
    g = tg.Grid(54, 54, 54, max_restart=1, device=DEV)
    rho = torch.rand(g.n_elem, dtype=torch.float64, device=DEV, generator=torch.Generator(DEV).manual_seed(3))
    v = torch.rand(g.n_dof, dtype=torch.float64, device=DEV, generator=torch.Generator(DEV).manual_seed(4))
    g.set_density(rho, 3.0, 1e-3)
    y = g.apply_K(v, tg.F64)
    with pytest.raises(TopoguardError):
        g.vcycle(v, tg.F64)
    g.set_density(rho, 3.0, 1e-3)
    assert torch.equal(g.apply_K(v, tg.F64), y) and torch.isfinite(y).all()


@pytest.mark.parametrize("n", [3, 17])
def test_setup_in_a_batch(n):
    dims = [(8, 4, 4), (64, 64, 32), (24, 12, 12), (16, 8, 8)]   # (a one-level grid changes its batch's sweeps)
    rng = np.random.default_rng(8)
    sel = [dims[i % 4] if i < 4 else dims[2 * (i % 2)] for i in range(n)]
    grids = [tg.Grid(*d, max_restart=3, device=DEV) for d in sel]
    rhos = [torch.tensor(rng.random(g.n_elem), device=DEV) for g in grids]
    print(f"setup of {n} problems", flush=True)
    b = tg.Batch(grids)
    b.set_density(rhos, 3.0, [1e-3] * n)
    fs = [torch.tensor(g.edge_load(), device=DEV) for g in grids]
    for prec in (tg.F64, tg.F32):
        opts = tg.solver_opts(prec=prec, max_iters=3, restart=3)
        us, _ = b.solve(fs, opts)
        for i, (d, r) in enumerate(zip(sel, rhos)):
            a = tg.Grid(*d, max_restart=3, device=DEV)
            a.set_density(r, 3.0, 1e-3)
            assert torch.equal(us[i], a.fgmres_solve(fs[i], opts)[0]), (d, prec)
