"""Build libgrpic.so in-tree with hipcc for gfx950.

Usage: python -m paper_2503_04558_amd.build

Each source is compiled to an object (in parallel) at -O3, then linked.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libgrpic.so")
OBJ = os.path.join(PKG, "_build")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    "-munsafe-fp-atomics",                       # hardware FP64 atomics (global and LDS)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed FP32 ops
    "-Wno-unused-command-line-argument",
]
# The reverse sweep's loops use more 64-bit constants than registers are left:
# formed where they are used, not ahead of the loops.  These are switches of the
# compiler's own; a compiler without them builds the source without them (more
# register spills, the same results).
SOURCE_FLAGS = {"adjoint.hip": ["-mllvm", "-disable-machine-licm", "-mllvm", "-amdgpu-use-amdgpu-trackers=1"]}


def sources() -> list[str]:
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    extra = SOURCE_FLAGS.get(os.path.basename(src), [])
    for flags in ([extra, []] if extra else [[]]):
        cmd = [HIPCC, "-O3", *FLAGS, *flags, "-I", INCLUDE, "-I", CSRC, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        rc = subprocess.call(cmd)
        if rc == 0:
            return obj
        if flags:
            print(f"{os.path.basename(src)}: not built with {' '.join(flags)}; without them", file=sys.stderr, flush=True)
    raise subprocess.CalledProcessError(rc, cmd)


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), sources()))
    cmd = [HIPCC, "--offload-arch=gfx950", "-fPIC", "-shared", *objs, "-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
