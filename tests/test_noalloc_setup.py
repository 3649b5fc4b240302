"""The no-allocation step sets up what its one launch reads, and no more.

The library runs on the CPU with counting stand-ins for the HIP calls
(``native/hip_calls.cpp``, preloaded): one launch, one occupancy query (of the
step kernel), and one copy for each table of the step (instances, smallest
cell sizes, patches, tiles, conservation-sum tiles) and for the Courant number.
"""

import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_1808_02638_amd", "libwavestep.so")

PROGRAM = r"""
import ctypes, sys
lib, stub, mx, my = sys.argv[1], sys.argv[2], int(sys.argv[3]), int(sys.argv[4])
class Patch(ctypes.Structure):
    _fields_ = [("mx", ctypes.c_int32), ("my", ctypes.c_int32), ("dx", ctypes.c_double),
                ("dy", ctypes.c_double), ("inst", ctypes.c_int32), ("bc", ctypes.c_int32)]
L, S = ctypes.CDLL(lib), ctypes.CDLL(stub)
mats = (ctypes.c_double * 2)(1.0, 4.0)
p = Patch(mx, my, 0.1, 0.1, 0, 1)
n, w = ctypes.c_int64(), ctypes.c_int64()
assert L.ws_layout(ctypes.byref(p), 1, 1, 0, ctypes.byref(n), ctypes.byref(w)) == 0
q = [ctypes.create_string_buffer(n.value) for _ in range(2)]
rc = L.ws_step_level_noalloc(ctypes.byref(p), 1, mats, 1, 0, 0, q[0], q[1], n,
                             ctypes.c_double(0.01), None, None)
assert rc == 0, rc
print(S.calls_of(0), S.calls_of(1), S.calls_of(2))
"""


@pytest.mark.parametrize("shape", [(64, 64), (400, 300)])
def test_one_step_sets_up_one_step(tmp_path, shape):
    stub = str(tmp_path / "hip_calls.so")
    subprocess.run(["g++", "-O1", "-fPIC", "-shared", "-o", stub,
                    os.path.join(HERE, "native", "hip_calls.cpp")], check=True)
    out = subprocess.run([sys.executable, "-c", PROGRAM, LIB, stub, *map(str, shape)],
                         env=dict(os.environ, LD_PRELOAD=stub), capture_output=True, text=True)
    assert out.returncode == 0, out.stderr
    copies, queries, launches = map(int, out.stdout.split())
    assert launches == 1
    assert queries == 1
    assert copies == 6
