"""The seed-row check when memory is short (CPU): gsrq_train_stage answers with a
status, no C++ exception leaves it."""
import os
import subprocess
import sys

import pytest

from paper_2607_01065_amd import gsrq as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = r"""
import ctypes, os, resource, sys
import numpy as np
from paper_2607_01065_amd import gsrq as B
lib = B.load_library()
N, K = int(sys.argv[1]), 65536
seeds = np.arange(K, dtype=np.int32)
seeds[-1] = 0 if sys.argv[2] == "twice" else seeds[-1]
sh = B.make_shape(N, 16, 16, K, 1)
need = ctypes.c_size_t()
assert lib.gsrq_train_workspace_bytes(ctypes.byref(sh), ctypes.byref(need)) == 0
one = 256   # stands for device memory: refused arguments never reach it
args = (ctypes.byref(sh), one, B.GSRQ_F32, 16, None, 1, seeds.ctypes.data, 0, one, one, None, None, None, None, one,
        0, None)
libc = ctypes.CDLL(None)
libc.malloc.restype = ctypes.c_void_p
pages = int(open("/proc/self/statm").read().split()[0])
resource.setrlimit(resource.RLIMIT_AS, (pages * os.sysconf("SC_PAGE_SIZE"),) * 2)
for size in (1 << 20, 1 << 17, 1 << 16):
    while libc.malloc(size):
        pass
os._exit(lib.gsrq_train_stage(*args))
"""


@pytest.mark.skipif(not os.path.exists(B.LIB_PATH), reason="libgsrq.so not built")
@pytest.mark.parametrize("N", [70000, (1 << 24) + 1])     # rows marked in a bit map; rows sorted
@pytest.mark.parametrize("seeds,status", [("distinct", B.GSRQ_E_WORKSPACE), ("twice", B.GSRQ_E_ARG)])
def test_seed_check_without_memory(N, seeds, status):
    r = subprocess.run([sys.executable, "-c", CHILD, str(N), seeds], cwd=ROOT, timeout=100, capture_output=True,
                       text=True)
    assert r.returncode == status, (r.returncode, r.stderr[-500:])
