"""An inner Krylov process on memory that held NaN: a zero right-hand side
stops it at once, gives a zero correction and leaves nothing behind that the
next process of the same memory reads.  The library's process functions are
called by their linker names; the operator is a diagonal in [1, 2], so GMRES
by least squares over its Krylov space is accurate to a few rounding errors of
the 2100-entry sums (1e-13), and 1e-11 leaves two orders."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2607_26382_amd import _lib

pytestmark = pytest.mark.gpu
CHUNK, PART_W = 2048, 256


class One(C.Structure):   # KrylovOne of tg_internal.h
    _fields_ = [("q", C.c_int), ("chunks", C.c_int), ("n", C.c_longlong), ("stride", C.c_longlong),
                ("sl", C.c_int * 12)] + [(k, C.c_void_p) for k in ("pool", "small", "part", "status", "list", "desc")]


def layout(q):
    """SmallLayout::init(q, q + 2)"""
    sizes = [(q + 1) * q, q + 1, q, q, q, PART_W, PART_W, 32, q + 3]
    o = [0]
    for s in sizes:
        o.append(o[-1] + s)
    return [q, q + 2] + o[:9] + [(o[9] + 31) & ~31]


@pytest.mark.parametrize("n,q", [(2100, 4), (2046, 1), (6000, 9)])
def test_zero_right_hand_side_leaves_nothing_behind(n, q):
    print(f"krylov stop n {n} q {q}", flush=True)
    lib = C.CDLL(_lib.lib()._name)
    S, D = C.c_void_p, C.c_void_p
    bind = lib._ZN2tg11krylov_bindERKNS_9KrylovOneEP12ihipStream_t
    start = lib._ZN2tg12krylov_startERKNS_9KrylovOneEPKdPdP12ihipStream_t
    step = lib._ZN2tg11krylov_stepERKNS_9KrylovOneEiP12ihipStream_t
    finish = lib._ZN2tg13krylov_finishERKNS_9KrylovOneEPdP12ihipStream_t
    chunks = -(-n // CHUNK)
    stride, sl = chunks * CHUNK, layout(q)

    def nan(k):
        return torch.full((k,), float("nan"), dtype=torch.float64, device="cuda")

    pool, small, part, status = nan((2 * q + 2) * stride), nan(sl[11]), nan((2 * q + 3) * chunks), nan(8)
    lst, desc = torch.zeros(2 * chunks, dtype=torch.int32, device="cuda"), nan(512)
    K = One(q, chunks, n, stride, (C.c_int * 12)(*sl), *(t.data_ptr() for t in (pool, small, part, status, lst, desc)))
    rows = pool.view(-1, stride)
    A = 1.0 + torch.rand(n, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    rr, out, stream = nan(1), nan(n), S(torch.cuda.current_stream().cuda_stream)

    def process(b):
        assert start(C.byref(K), D(b.data_ptr()), D(rr.data_ptr()), stream) == 0
        for j in range(q):
            rows[q + 2 + j, :n] = rows[j, :n] * small[sl[9] + 8]   # z = v / rho
            rows[q + 1, :n] = A * rows[q + 2 + j, :n]
            assert step(C.byref(K), j, stream) == 0
        assert finish(C.byref(K), D(out.data_ptr()), stream) == 0
        return out.clone()

    assert bind(C.byref(K), stream) == 0
    assert torch.count_nonzero(process(torch.zeros(n, dtype=torch.float64, device="cuda"))) == 0
    b = torch.randn(n, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    x = process(b).cpu().numpy()
    a, bn = A.cpu().numpy(), b.cpu().numpy()
    Z = np.linalg.qr(np.stack([bn * np.cos(j * np.arccos(2 * a - 3)) for j in range(q)], axis=1))[0]   # the Krylov space
    ref = Z @ np.linalg.lstsq(a[:, None] * Z, bn, rcond=None)[0]
    assert np.linalg.norm(x - ref) <= 1e-11 * np.linalg.norm(ref)
