"""Build the HIP library liblbmhd.so in-tree for gfx950 with hipcc.

hipcc cross-compiles without a GPU, so this runs anywhere ROCm is installed.
Usage: ``python -m paper_1705_09807_amd.build`` or ``build()``.
"""

from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "liblbmhd.so")

SOURCES = ["lbmhd_kernels.hip", "lbmhd_steps_fp64.hip", "lbmhd_steps_fp32.hip", "lbmhd_steps_16bit.hip", "lbmhd_inplace.hip",
           "lbmhd_learned.hip", "lbmhd_spectra.hip", "lbmhd_shape.cpp", "lbmhd_plan.cpp",
           "lbmhd_api.cpp"]

# Packed FP32 instructions are disabled for all device code; the host pass
# warns that it does not know the feature, which is harmless.
FLAGS = [
    "-O3",
    "-std=c++17",
    "--offload-arch=gfx950",
    "-fPIC",
    "-Wall",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def hipcc() -> str:
    path = os.environ.get("HIPCC") or shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(path):
        raise RuntimeError("hipcc not found; a ROCm installation is required to build liblbmhd.so")
    return path


def _run(cmd, verbose: bool):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed building liblbmhd.so")
    if verbose and res.stderr.strip():
        sys.stderr.write(res.stderr)


def build(verbose: bool = False) -> str:
    """Compile csrc/ into liblbmhd.so (always recompiles; the sources side by side).
    Returns its path."""
    tmp = LIB + ".tmp"
    cc = hipcc()
    with tempfile.TemporaryDirectory() as work:
        objs = [os.path.join(work, s + ".o") for s in SOURCES]
        with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
            jobs = [pool.submit(_run, [cc, *FLAGS, "-I", INCLUDE, "-I", CSRC, "-c", os.path.join(CSRC, s), "-o", o],
                                verbose) for s, o in zip(SOURCES, objs)]
            for job in jobs:
                job.result()
        _run([cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
