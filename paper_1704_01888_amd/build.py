"""Build libpa.so (HIP for gfx950) in the package directory."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libpa.so")
# (source, extra flags); pa_kernels.hip comes before the other kernels, so that
# its code object is the first of the library's
UNITS = [("pa_host.cpp", []), ("pa_kernels.hip", []), ("pa_probe.hip", []), ("pa_static.hip", []),
         *[("pa_quad_any.hip", [f"-DPA_PART={i}"]) for i in range(4)]]

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    # no packed FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-ffp-contract=off",
    "-Wall",
]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)


def build(verbose: bool = False) -> str:
    """Compile the units side by side and link them."""
    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as d, ThreadPoolExecutor(min(len(UNITS), os.cpu_count() or 1)) as pool:
        objs = [os.path.join(d, f"{i}.o") for i in range(len(UNITS))]
        jobs = [pool.submit(_run, ["hipcc", *HIPCC_FLAGS, *flags, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                                   "-c", "-o", obj, os.path.join(CSRC, src)], verbose)
                for obj, (src, flags) in zip(objs, UNITS)]
        for j in jobs:
            j.result()
        _run(["hipcc", "--offload-arch=gfx950", "-fPIC", "-shared", "-o", tmp, *objs], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
