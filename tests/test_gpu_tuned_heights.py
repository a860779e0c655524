"""Heights from the autotuner stay in use while the running problems fill the
device at them, and give way to the rule's below 1024 tiles.  600 grids of
16x8x8 (9 node layers, 2 tiles each at the cached height 9): 1198 tiles when one
problem stopped, 600 when half of them did, where the rule gives 5 layers.  The
heights are read through the linker names of the library's batch functions, in
a process of its own, since the cache file is read once."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import ctypes as C
from paper_2607_26382_amd import _lib, topoguard as tg
N = 600
grids = [tg.Grid(16, 8, 8, max_restart=1, device="cuda") for _ in range(N)]
b = tg.Batch(grids)
lib = C.CDLL(_lib.lib()._name)
def height(active):
    a = (C.c_int * len(active))(*active)
    vec = (C.c_void_p * 3)(C.addressof(a), C.addressof(a) + C.sizeof(a), C.addressof(a) + C.sizeof(a))
    assert lib._ZN2tg16batch_set_activeEPNS_5BatchERKSt6vectorIiSaIiEEP12ihipStream_tb(b.handle, vec, None, False) == 0
    return lib._ZN2tg12batch_zc_runEPKNS_5BatchEii(b.handle, active[0], 0)
every = list(range(N))
rule = [height(every), height(every[1:]), height(every[::2])]
b.autotune(tg.F32)   # from the file
print("heights", *rule, height(every), height(every[1:]), height(every[::2]), height(every), flush=True)
"""


def test_tuned_heights_outlive_the_first_stop(tmp_path):
    cache = tmp_path / "heights"
    cache.write_text("p1_n600_600x16.8.8 8 9 0 0 0 0 0 0 0\n")
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, env={**os.environ, "TG_AUTOTUNE_CACHE": str(cache)},
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    heights = [int(x) for x in r.stdout.split("heights")[1].split()]
    assert heights[:2] == [8, 8]                   # the rule: 2048 tiles at 8 (5 balanced)
    assert heights[3:] == [9, 9, heights[2], 9] and heights[2] < 9
