"""Build libmdot.so (HIP, gfx950) in-tree with hipcc.

Every HIP source is compiled with `-Xclang -target-feature -Xclang -packed-fp32-ops`
so the compiler does not form packed FP32 instructions; the hot loops are written with
scalar FP32/FP64 arithmetic.
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT_DIR = os.path.join(HERE, "_lib")
LIB = os.path.join(OUT_DIR, "libmdot.so")
SOURCES = ["mdot_kernels.hip", "mdot_api.cpp"]
ARCH = os.environ.get("MDOT_OFFLOAD_ARCH", "gfx950")


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def build(verbose: bool = False) -> str:
    os.makedirs(OUT_DIR, exist_ok=True)
    objs = []
    common = ["-O3", "-std=c++17", "-fPIC", f"-I{os.path.join(ROOT, 'include')}", "-Wall",
              "-Wno-unused-function"]
    for src in SOURCES:
        path = os.path.join(CSRC, src)
        obj = os.path.join(OUT_DIR, src + ".o")
        cmd = [hipcc(), *common, "-c", path, "-o", obj]
        if src.endswith(".hip"):
            # kernel arguments (a few pointers and ints) are preloaded into SGPRs at dispatch, so a
            # kernel's first dependent load does not wait for a kernarg-segment fetch
            cmd += [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-munsafe-fp-atomics", "-mllvm", "-amdgpu-kernarg-preload-count=16",
                    # the constants of exp and log stay where they are used: hoisted out of the loops of
                    # the resident kernels they take 30 to 80 registers and spill (k_steps on FP32 costs 256
                    # and 21 to 28 spilled, now 220 to 225 and none; on clouds 128 and 26 to 46, now 108 to
                    # 124 and none). k_fin falls from 232 and 256 registers to 194 and 226; sweeps keep
                    # theirs within 3
                    "-mllvm", "-disable-machine-licm"]
        else:
            pass
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        objs.append(obj)
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
