"""A grid whose density came through a batch, used alone: operator, V-cycle,
adaptive stack and spectrum read the density of that batch.  The set-up is the
same for a problem alone and in a batch and so are the single-grid calls, so
every result is compared bit for bit with a grid that set the density itself.
Also after the grid is bound anew, and after a second density through a second
batch."""
import pytest
import torch

from paper_2607_26382_amd import synth
from paper_2607_26382_amd import topoguard as tg

pytestmark = pytest.mark.gpu
DEV = "cuda"


def alone(g, v):
    out = [g.apply_K(v), g.vcycle(v), g.apply_K(v.float(), tg.BF16X3MFMA), g.vcycle(v.float(), tg.BF16X3MFMA)]
    out.append(g.stack_precondition(v)[0])
    out.append(torch.tensor([float(x) for x in g.extreme_eigenvalues(max_iters=6).values() if isinstance(x, float)]))
    return out


@pytest.mark.parametrize("dims", [((8, 4, 4), (16, 8, 8)), ((32, 16, 16), (16, 8, 8), (32, 16, 16))])
def test_single_grid_calls_see_the_batch_density(dims):
    print(f"density by batch {dims}", flush=True)
    grids = [tg.Grid(*d, max_restart=5, device=DEV) for d in dims]
    twins = [tg.Grid(*d, max_restart=5, device=DEV) for d in dims]
    batches = [tg.Batch(grids), tg.Batch(grids[::-1])]

    def check(batch, order, seed, floor):
        rhos = [torch.tensor(synth.uniform(*d, seed + i), device=DEV) for i, d in enumerate(dims)]
        batch.set_density([rhos[i] for i in order], 3.0, [floor] * len(dims))
        for g, t, r, d in zip(grids, twins, rhos, dims):
            t.set_density(r, 3.0, floor)
            v = torch.randn(t.n_dof, dtype=torch.float64, device=DEV, generator=torch.Generator(DEV).manual_seed(seed))
            v.view(d[2] + 1, d[1] + 1, d[0] + 1, 3)[:, :, 0] = 0.0
            for a, b in zip(alone(g, v), alone(t, v)):
                assert torch.equal(a, b)

    order = list(range(len(dims)))
    check(batches[0], order, 1, 1e-3)
    check(batches[1], order[::-1], 5, 1e-2)
    grids[0].bind(DEV)
    check(batches[0], order, 9, 1e-3)
