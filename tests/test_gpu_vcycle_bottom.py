"""The one-launch bottom of the V-cycle: the workgroup of a problem and its
helpers are found from the launch's index, and how many helpers there are
depends on the number of problems (none from 129 on).  A problem's result is
the same, bit for bit, alone and anywhere in a batch of any size, and the cycle
agrees with the oracle's where the level sizes leave remainders of the
workgroup: more nodes than threads, coarse levels of odd sizes, a coarsest
system longer than the entries read ahead.  Tolerances as for the V-cycle's
other comparisons."""
import numpy as np
import pytest
import torch

from oracle import ke as oke, mesh, multigrid as omg, operator as op
from paper_2607_26382_amd import topoguard as tg

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("prec", [tg.F64, tg.F32, tg.BF16X3MFMA])
@pytest.mark.parametrize("n", [2, 9, 57, 130])
def test_same_alone_and_in_batches(n, prec):
    dims = [(8, 4, 4), (16, 8, 8), (12, 4, 8)]
    print(f"bottom: {n} problems, precision {prec}", flush=True)
    opts = tg.solver_opts(prec=prec, max_iters=12, restart=12)
    rng = np.random.default_rng(11)
    rho = [torch.tensor(rng.random(d[0] * d[1] * d[2]), device=DEV) for d in dims]
    alone, load = [], []
    for d, r in zip(dims, rho):
        g = tg.Grid(*d, max_restart=12, device=DEV)
        g.set_density(r, 3.0, 1e-3)
        load.append(torch.tensor(g.edge_load(), device=DEV))
        alone.append(g.fgmres_solve(load[-1], opts))
    grids = [tg.Grid(*dims[i % 3], max_restart=12, device=DEV) for i in range(n)]
    b = tg.Batch(grids)
    b.set_density([rho[i % 3] for i in range(n)], 3.0, [1e-3] * n)
    us, res = b.solve([load[i % 3] for i in range(n)], opts)
    for i in range(n):
        assert res[i]["iterations"] == alone[i % 3][1]["iterations"], i
        assert torch.equal(us[i], alone[i % 3][0]), i


@pytest.mark.parametrize("dims", [(24, 12, 12), (40, 16, 24), (64, 32, 32), (12, 8, 12)])
def test_cycle_matches_oracle(dims):
    print(f"bottom: cycle {dims}", flush=True)
    rng = np.random.default_rng(5)
    og = mesh.Grid(*dims)
    rho, free = rng.random(og.n_elem), og.free_dofs()
    H = omg.build_hierarchy(og, op.young(rho, 3.0, 1e-3), oke.ke())
    g = tg.Grid(*dims, max_restart=1, device=DEV)
    g.set_density(torch.tensor(rho, device=DEV), 3.0, 1e-3)
    r = np.zeros(og.n_dof)
    r[free] = rng.standard_normal(int(free.sum()))
    ref = omg.vcycle(H, r[free])
    for prec, tol in ((tg.F64, 1e-9), (tg.F32, 2e-3), (tg.BF16X3MFMA, 2e-3)):
        z = g.vcycle(torch.tensor(r, device=DEV, dtype=torch.float64 if prec == tg.F64 else torch.float32), prec)
        z = z.double().cpu().numpy()
        assert np.all(z[~free] == 0.0)
        assert np.abs(z[free] - ref).max() <= tol * np.abs(ref).max()
