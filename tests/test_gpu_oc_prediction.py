"""The multiplier's bisection where the predicted way through it is bad: volumes
that are flat or jump between clipped designs, sensitivities that are zero for
half of the elements, a steep projection, a bracket whose upper end is still
the initial 1e9.  The halvings decide as one at a time whatever is predicted:
the oracle's multiplier to the bisection's relative width (1e-9), and its design."""
import numpy as np
import pytest
import torch

from oracle import mesh, topopt as to
from paper_2607_26382_amd import topoguard as tg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(16, 8, 8), (80, 60, 60)])     # seven and three midpoints a launch
@pytest.mark.parametrize("field,move,beta,scale", [
    ("two", 0.05, 1.0, 1.0), ("half", 0.2, 4.0, 1e-3), ("wide", 0.2, 8.0, 1.0), ("wide", 1e-3, 1.0, 1e-6),
    ("wide", 0.2, 1.0, 3e8)])
def test_multiplier_equals_oracle(dims, field, move, beta, scale):
    print(f"multiplier {dims} {field} move {move} beta {beta} scale {scale}", flush=True)
    rng = np.random.default_rng(12)
    og = mesh.Grid(*dims)
    g = tg.Grid(*dims, max_restart=1, device="cuda")
    n = og.n_elem
    x = 0.3 + 0.2 * (rng.random(n) - 0.5)
    q = rng.random(n)
    dc = -scale * {"two": np.where(q < 0.4, 1.0, 100.0), "half": np.where(q < 0.5, 0.0, q), "wide": np.exp(12 * q)}[field]
    dv = np.ones(n)
    t = lambda a: torch.tensor(a, device="cuda")
    xn, lam = g.oc_update(t(x), t(dc), t(dv), 0.3, move, 0.9, beta)
    xr, lr = to.oc_update(og, x, dc, dv, 0.3, move, 0.9, beta)
    assert lam == pytest.approx(lr, rel=2e-9)
    assert np.abs(xn.cpu().numpy() - xr).max() <= 1e-9
