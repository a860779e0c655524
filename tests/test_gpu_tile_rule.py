"""The z-tile height rule in each of its regimes: one small grid (a layer per
tile), as many tiles as the 768 allow, the 2048-tile regime and tall grids.
The heights only split the work, so a problem of the batch solves bit for bit
as it does alone, where the rule gives other heights."""
import pytest
import torch

from paper_2607_26382_amd import synth
from paper_2607_26382_amd import topoguard as tg

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dims,count,height", [((16, 8, 8), 1, 1), ((32, 16, 16), 40, 6), ((32, 16, 16), 130, 6),
                                               ((64, 32, 32), 24, 6), ((16, 16, 64), 70, 22)])
def test_heights_and_equal_bits(dims, count, height):
    rhos = [torch.tensor(synth.uniform(*dims, s), device=DEV) for s in range(count)]
    grids = [tg.Grid(*dims, max_restart=3, device=DEV) for _ in range(count)]
    f = torch.tensor(grids[0].edge_load(), device=DEV)
    b = tg.Batch(grids)
    assert b.tile_heights(0)[0] == height
    b.set_density(rhos, 3.0, [1e-3] * count)
    for prec in (tg.BF16X3MFMA, tg.F64):
        o = tg.solver_opts(prec=prec, restart=3, max_iters=3, tol=0.0)
        us, _ = b.solve([f] * count, o)
        one = tg.Grid(*dims, max_restart=3, device=DEV)
        for i in {0, count - 1}:
            one.set_density(rhos[i], 3.0, 1e-3)
            u, _, _ = one.fgmres_solve(f, o)
            assert torch.equal(u, us[i])
