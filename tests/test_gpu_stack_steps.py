"""The full adaptive stack where its launches change: every Chebyshev degree
from one (the first two steps of a zero start are one launch, the third reads
a kept iterate; the first step after the coarse correction prolongs it), the
levels that one workgroup holds and those stepped from the host, inner
processes of one step, of the longest that the batched kernels take and one
longer, and no scale, one scale and several before a coarse V-cycle.

One application on two seeded vectors against the oracle.  The comparison is
between two FP64 computations of the same map: its differences are rounding
times the conditioning of the inner least squares (some 1e-10 here), so 1e-7
of the output's norm, as for the default stack, leaves two orders."""
import numpy as np
import pytest
import torch

from oracle import adaptive as oad
from oracle import ke as oke
from oracle import mesh
from oracle import multigrid as omg
from oracle import operator as op
from paper_2607_26382_amd import synth
from paper_2607_26382_amd import topoguard as tg

pytestmark = pytest.mark.gpu

# dims, nu_pre, nu_post, coarse_steps, inner_steps; 8x4x4 has two levels,
# 16x8x8 and 24x12x8 three (level 1 is held by one workgroup), 32x16x16 four
# (level 1 is stepped, level 2 held)
CASES = [
    ((8, 4, 4), 1, 1, 0, 1), ((8, 4, 4), 3, 2, 4, 126), ((8, 4, 4), 2, 4, 1, 127),
    ((16, 8, 8), 1, 1, 1, 1), ((16, 8, 8), 2, 1, 0, 2), ((16, 8, 8), 4, 3, 7, 9),
    ((24, 12, 8), 1, 3, 2, 0), ((24, 12, 8), 5, 1, 3, 21),
    ((32, 16, 16), 1, 1, 2, 3), ((32, 16, 16), 2, 3, 1, 2), ((32, 16, 16), 3, 1, 0, 1), ((32, 16, 16), 4, 4, 3, 5),
]


@pytest.mark.parametrize("dims,pre,post,coarse,inner", CASES)
def test_application_matches_oracle(dims, pre, post, coarse, inner):
    print(f"stack steps {dims} degrees {pre}/{post} coarse {coarse} inner {inner}", flush=True)
    rho = synth.blobs(*dims, 7, blob=4)
    og = mesh.Grid(*dims)
    free = og.free_dofs()
    H = omg.build_hierarchy(og, op.young(rho, 3.0, 1e-3), oke.ke())
    g = tg.Grid(*dims, device="cuda")
    g.set_density(torch.tensor(rho, dtype=torch.float64, device="cuda"), 3.0, 1e-3)
    so = tg.stack_opts(nu_pre=pre, nu_post=post, coarse_steps=coarse, inner_steps=inner)
    M = oad.adaptive_stack(H, inner_steps=inner, coarse_steps=coarse, theta=so.theta, nu_pre=pre, nu_post=post,
                           lo=so.lo, hi=so.hi)
    rng = np.random.default_rng(3)
    for _ in range(2):
        v = np.zeros(og.n_dof)
        v[free] = rng.standard_normal(int(free.sum()))
        ref = M(v[free])
        _, _, ok, kept = M.log[-1]
        z, lg = g.stack_precondition(torch.tensor(v, device="cuda"), so)
        z = z.cpu().numpy()
        assert lg["coarse_accepted"] == ok and lg["fine_kept"] == kept
        assert np.all(z[~free] == 0.0)
        assert np.linalg.norm(z[free] - ref) <= 1e-7 * np.linalg.norm(ref)
