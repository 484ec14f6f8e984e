"""Build libsgn.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2506_16045_amd.build          # or build() from Python

The library is a plain C-ABI shared object (include/sgn.h); no PyTorch headers
are involved.  Packed FP32 instructions are disabled for every HIP source.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libsgn.so")
SOURCES = ["sgn_lib.hip", "sgn_line_solve.hip", "sgn_line_rk4.hip", "sgn_line_rk4_mixed.hip", "sgn_line_linimp.hip", "sgn_server.hip"]
ARCH = os.environ.get("SGN_OFFLOAD_ARCH", "gfx950")


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build libsgn.so)")


def flags():
    return [
        f"--offload-arch={ARCH}",
        "-O3",
        "-std=c++17",
        "-fPIC",
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-I", INCLUDE,
        "-I", CSRC,
        "-Wall", "-Wno-unused-function", "-Wno-unused-variable", "-Wno-unused-parameter",
    ]


def build(verbose: bool = True) -> str:
    objs, running = [], []
    for src in SOURCES:   # side by side: one compiler process per source
        obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc(), *flags(), "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        running.append((cmd, subprocess.Popen(cmd)))
        objs.append(obj)
    codes = [(cmd, p.wait()) for cmd, p in running]
    for cmd, rc in codes:
        if rc:
            raise subprocess.CalledProcessError(rc, cmd)
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    for o in objs:
        os.remove(o)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    print(LIB)
    sys.exit(0)
