"""Build libsse.so (every HIP source under csrc/) for gfx950 with hipcc."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libsse.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# Packed fp32 VALU ops stay off: hipcc would otherwise form them from float2 code.
# The atomic optimizer stays off too: the persistent kernels' tile pull is a
# single-lane atomic whose result is needed only when the current tile ends, and
# the optimizer's wave-reduced form reads the result back at once.
HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
             "-Wno-unused-command-line-argument"]


def sources():
    return sorted(glob.glob(os.path.join(PKG, "csrc", "*.hip")))


def build(verbose: bool = False, extra=()) -> str:
    """Compile the sources side by side to objects in _build/, link libsse.so in the package."""
    bdir = os.path.join(ROOT, "_build")
    os.makedirs(bdir, exist_ok=True)
    cmds, objs = [], []
    for src in sources():
        objs.append(os.path.join(bdir, os.path.basename(src) + ".o"))
        cmds.append([HIPCC, *HIP_FLAGS, *extra, "-I", os.path.join(ROOT, "include"),
                     "-I", os.path.join(PKG, "csrc"), "-c", src, "-o", objs[-1]])
        if verbose:
            print(" ".join(cmds[-1]), flush=True)
    with ThreadPoolExecutor(min(8, len(cmds))) as pool:
        list(pool.map(lambda c: subprocess.run(c, check=True), cmds))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
