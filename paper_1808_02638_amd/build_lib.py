"""Build the gfx950 shared library ``libwavestep.so`` in-tree with hipcc."""

from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
# (source, object, extra flags): the step kernels compile in seven parts
SOURCES = [("ws_kernels.hip", f"ws_kernels_{n}.o", [f"-DWS_PART={n}"]) for n in range(7)] + [
    (f"ws_{n}.hip", f"ws_{n}.o", []) for n in ("multi", "block", "adjoint", "amr", "api")]
LIB = os.path.join(HERE, "libwavestep.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-ffp-contract=off",  # every cell's arithmetic is fixed by the source
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-unused-function",  # a part of the step kernels uses some of the file's helpers
]


def build(verbose: bool = False) -> str:
    """Compile every source (in parallel, one hipcc each) and link the library."""
    objs, procs = [], []
    for src, name, extra in SOURCES:
        obj = os.path.join(CSRC, name)
        cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((cmd, subprocess.Popen(cmd)))
        objs.append(obj)
    failed = [cmd for cmd, p in procs if p.wait() != 0]
    if failed:
        raise subprocess.CalledProcessError(1, failed[0])
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    for o in objs:
        os.remove(o)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
