"""tg_vcycle on external vectors: the first two sweeps read the input and the
last writes the output directly where every grid has at least two levels and
nu_pre >= 2, and go through copies otherwise.  Every form against the oracle's
V-cycle: one and several levels, each precision, one and more sweeps, and the
output over the input.  Tolerances as for the V-cycle's other comparisons:
1e-9 of the largest entry in FP64, 2e-3 in FP32 with BF16 products in split
form."""
import numpy as np
import pytest
import torch

from oracle import ke as oke, mesh, multigrid as omg, operator as op
from paper_2607_26382_amd import topoguard as tg

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("nu_pre,nu_post", [(2, 2), (1, 1), (1, 2), (3, 1)])
@pytest.mark.parametrize("dims", [(4, 2, 2), (16, 8, 8), (12, 8, 12)])
def test_vcycle_external_vectors(dims, nu_pre, nu_post):
    rng = np.random.default_rng(7)
    og = mesh.Grid(*dims)
    rho, free = rng.random(og.n_elem), og.free_dofs()
    H = omg.build_hierarchy(og, op.young(rho, 3.0, 1e-3), oke.ke())
    g = tg.Grid(*dims, mg=tg.mg_opts(nu_pre=nu_pre, nu_post=nu_post), max_restart=1, device=DEV)
    g.set_density(torch.tensor(rho, device=DEV), 3.0, 1e-3)
    r = rng.standard_normal(og.n_dof)          # clamped entries not zero: they are ignored
    ref = omg.vcycle(H, r[free], nu_pre=nu_pre, nu_post=nu_post)
    for prec, tol in ((tg.F64, 1e-9), (tg.F32, 2e-3), (tg.BF16X3MFMA, 2e-3)):
        v = torch.tensor(r, device=DEV, dtype=torch.float64 if prec == tg.F64 else torch.float32)
        z = g.vcycle(v, prec)
        zc = z.double().cpu().numpy()
        assert np.all(zc[~free] == 0.0)
        assert np.abs(zc[free] - ref).max() <= tol * np.abs(ref).max()
        # the output may be the input
        tg.check(tg.lib().tg_vcycle(g.handle, tg._ptr(v), tg._ptr(v), prec, tg._stream()))
        assert torch.equal(v, z)
