"""The prolonging sweep at the tallest tile that takes it, 14 layers, and the
first height above, 15, where the prolongation is a pass of its own: the
problem of a batch solves bit for bit as it does alone, at tiles of one layer.
The heights are the rule's: the tallest that still gives 2048 tiles, balanced."""
import numpy as np
import pytest
import torch

from paper_2607_26382_amd import topoguard as tg

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("prec", [tg.F64, tg.F32, tg.BF16X3MFMA])
@pytest.mark.parametrize("dims,n,height", [((16, 16, 40), 180, 14), ((16, 16, 28), 260, 15)])
def test_limit_of_the_prolonging_sweep(dims, n, height, prec):
    print(f"prolong limit {dims} height {height} precision {prec}", flush=True)
    rng = np.random.default_rng(8)
    rho = [torch.tensor(rng.random(int(np.prod(dims))), device=DEV) for _ in range(2)]
    opts = tg.solver_opts(prec=prec, max_iters=3, restart=3)
    alone = []
    for r in rho:
        g = tg.Grid(*dims, max_restart=3, device=DEV)
        g.set_density(r, 3.0, 1e-3)
        f = torch.tensor(g.edge_load(), device=DEV)
        alone.append(g.fgmres_solve(f, opts)[0])
    b = tg.Batch([tg.Grid(*dims, max_restart=3, device=DEV) for _ in range(n)])
    assert b.tile_heights(0)[0] == height
    b.set_density([rho[i % 2] for i in range(n)], 3.0, [1e-3] * n)
    us, _ = b.solve([f] * n, opts)
    for i in range(n):
        assert torch.equal(us[i], alone[i % 2]), i
