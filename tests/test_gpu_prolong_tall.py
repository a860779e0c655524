"""The post-sweep that prolongs, on tall z tiles: batches that fill the device
get heights of 6 to 13 layers at the finest level, up to the tallest (14) that
form x + P e themselves, and every problem's result is the same, bit for bit,
as alone, where its tiles are a layer or two."""
import numpy as np
import pytest
import torch

from paper_2607_26382_amd import topoguard as tg

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("prec", [tg.F64, tg.F32, tg.BF16X3MFMA])
@pytest.mark.parametrize("n", [60, 120, 180, 320])
def test_batch_of_tall_tiles_equals_alone(n, prec):
    dims = (16, 16, 48)
    rng = np.random.default_rng(6)
    rho = [torch.tensor(rng.random(16 * 16 * 48), device=DEV) for _ in range(3)]
    opts = tg.solver_opts(prec=prec, max_iters=3, restart=3)
    alone = []
    for r in rho:
        g = tg.Grid(*dims, max_restart=3, device=DEV)
        g.set_density(r, 3.0, 1e-3)
        f = torch.tensor(g.edge_load(), device=DEV)
        alone.append(g.fgmres_solve(f, opts)[0])
    b = tg.Batch([tg.Grid(*dims, max_restart=3, device=DEV) for _ in range(n)])
    b.set_density([rho[i % 3] for i in range(n)], 3.0, [1e-3] * n)
    us, _ = b.solve([f] * n, opts)
    print(f"tall tiles: {n} problems, precision {prec}, heights {b.tile_heights(0)}", flush=True)
    for i in range(n):
        assert torch.equal(us[i], alone[i % 3]), i
