"""The operator of a lone grid takes tile heights of its own, one per
arithmetic; the sum at a node does not depend on them, so every result is
compared bit for bit with the same problem's in a batch, which takes the sweeps'
height.  Grids of one tile, of an odd rest in every dimension, and of the
sizes where the own heights are the lowest, in between and tall."""
import ctypes as C

import pytest
import torch

from paper_2607_26382_amd import _lib
from paper_2607_26382_amd import synth
from paper_2607_26382_amd import topoguard as tg

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dims", [(1, 1, 1), (3, 2, 2), (14, 14, 16), (29, 31, 15), (74, 44, 45), (99, 68, 44),
                                  (96, 40, 97), (150, 104, 70)])
@pytest.mark.parametrize("prec", [tg.F64, tg.F32, tg.BF16MFMA, tg.BF16X3MFMA])
def test_own_heights_give_the_batch_bits(dims, prec):
    print(f"lone operator {dims} precision {prec}", flush=True)
    rho = torch.tensor(synth.uniform(*dims, 3), device=DEV)
    g = tg.Grid(*dims, max_restart=1, device=DEV)
    g.set_density(rho, 3.0, 1e-3)
    u = torch.randn(g.n_dof, dtype=torch.float64, device=DEV, generator=torch.Generator(DEV).manual_seed(2))
    u = u if prec == tg.F64 else u.float()
    y = g.apply_K(u, prec)
    # a batch's heights on the same grid: the operator's tile list, by the library's linker names
    lib = C.CDLL(_lib.lib()._name)
    pair = tg.Batch([g, tg.Grid(*dims, max_restart=1, device=DEV)])
    one = (C.c_int * 1)(0)
    vec = (C.c_void_p * 3)(C.addressof(one), C.addressof(one) + 4, C.addressof(one) + 4)
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert lib._ZN2tg16batch_set_activeEPNS_5BatchERKSt6vectorIiSaIiEEP12ihipStream_tb(pair.handle, vec, stream,
                                                                                        False) == 0
    z = torch.full_like(u, float("nan"))
    assert lib._ZN2tg7k_applyEPNS_5BatchEiiPKviPvP12ihipStream_t(pair.handle, prec, -1, C.c_void_p(u.data_ptr()), -1,
                                                                 C.c_void_p(z.data_ptr()), stream) == 0
    assert torch.equal(y, z)
