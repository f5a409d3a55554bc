"""Host side of the bond-table set-up (no GPU needed: the tables are made
before the first device call): the tables of the shared draws, and what
happens when the host runs out of memory, with the library's allocations
bounded by the address space left to a child process."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PYRO_ENOMEM, PYRO_EDEVICE = -2, -3

CHILD = r"""
import ctypes, os, resource, sys
import numpy as np
sys.path.insert(0, sys.argv[1])
os.environ["HIP_VISIBLE_DEVICES"] = ""  # the set-up ends at its first device call
from paper_1612_08312_amd import pyrosw
lib = pyrosw.load_library()
n, nb = 1 << 22, 16 << 20
a = (np.arange(nb, dtype=np.int64) // 4).astype(np.int32)  # in windows of their own, 16 to a block
b = a ^ 1
h = ctypes.c_void_p()
page = os.sysconf("SC_PAGE_SIZE")
size = int(open("/proc/self/statm").read().split()[0]) * page
limit = size + int(float(sys.argv[2]) * (1 << 20))
resource.setrlimit(resource.RLIMIT_AS, (limit, limit))
p = ctypes.POINTER(ctypes.c_int32)
rc = lib.pyro_sw_graph_init(ctypes.byref(h), ctypes.c_int64(n), ctypes.c_int64(nb), a.ctypes.data_as(p),
                            b.ctypes.data_as(p), ctypes.c_int(1), ctypes.c_double(2.0), ctypes.c_double(1.0),
                            ctypes.c_uint64(1), ctypes.c_int(1), ctypes.c_void_p(None))
print("rc", rc, flush=True)
os._exit(0)
"""


# The bond arrays take 192 MiB, the window positions 64, the draws 32 and more.
@pytest.mark.parametrize("mib", [40, 100, 150, 215, 240, 262, 275, 290])
def test_set_up_survives_any_shortage(mib):
    r = subprocess.run([sys.executable, "-c", CHILD, ROOT, str(mib)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (mib, r.returncode, r.stderr[-500:])
    rc = int(r.stdout.split()[1])
    assert rc in (PYRO_ENOMEM, PYRO_EDEVICE), (mib, rc)


def test_draw_tables(tmp_path):
    exe = str(tmp_path / "draws_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_1612_08312_amd", "csrc"),
                    os.path.join(ROOT, "tests", "draws_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "draws ok" in r.stdout, r.stderr
