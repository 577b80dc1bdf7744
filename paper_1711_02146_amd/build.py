"""Build libpa.so (HIP kernels + C-ABI host code) for gfx950 with hipcc.

    python -m paper_1711_02146_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libpa.so")
SOURCES = ["pa_kernels.hip", "pa_host.cpp", "pa_batch.cpp", "pa_stepper.cpp", "pa_tune.cpp"]
# pa_kernels.hip includes pa_real_kernels.inc (the real-coupling kernels); it is
# also compiled once per lattice size for the kernels instantiated per L
KERNEL_LS = (4, 6, 8, 10, 12, 14, 16)

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-ffp-contract=off",          # host FP64 table: every line rounds as written
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-pass-failed",           # partial unroll hints on loops with a run-time start
    "-I" + os.path.join(ROOT, "include"),
]


def build(verbose: bool = False) -> str:
    units = [(src, src.rsplit(".", 1)[0] + ".o", []) for src in SOURCES]
    # the slowest first: the objects are compiled in parallel
    units = [("pa_kernels.hip", f"pa_kernels_L{L}.o", [f"-DPA_KERNEL_L={L}"])
             for L in reversed(KERNEL_LS)] + units

    def compile_unit(unit):
        src, obj, defs = unit
        obj = os.path.join(CSRC, obj)
        if defs:  # an object of one lattice size leaves the file's other kernels unused
            defs = [*defs, "-Wno-unused-function", "-Wno-unneeded-internal-declaration"]
        elif src == "pa_kernels.hip":
            defs = ["-Wno-unneeded-internal-declaration"]
        cmd = [HIPCC, *FLAGS, *defs, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
        objs = list(pool.map(compile_unit, units))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
