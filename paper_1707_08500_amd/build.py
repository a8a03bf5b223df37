"""Builds libpsatd.so (HIP, gfx950 only) in-tree next to this file.

    python -m paper_1707_08500_amd.build

The library is the whole product path; the Python binding only marshals
arguments into it.
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libpsatd.so")

# (source, defines): the kernels are compiled as one translation unit per
# precision form (psatd_kernels.hip, PSATD_TU), all units at once
UNITS = [("psatd_api.hip", [])] + [("psatd_kernels.hip", [f"-DPSATD_TU={i}"]) for i in range(5)]
SOURCES = ["psatd_api.hip", "psatd_kernels.hip"]
HEADERS = ["fft_engine.hpp", "psatd_device.hpp", "psatd_launch.hpp", "plan_host.hpp", "dft_consts.h",
           "mfma_dft.hpp", "reg_fft.hpp", "zreg.hpp"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # hand-written code only: keep the compiler from forming packed FP32 ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-unused-function",
    "-Wno-unused-variable",
]


def build(verbose: bool = True) -> str:
    """Compiles every HIP source into libpsatd.so; returns its path."""
    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as obj:
        jobs, objs = [], []
        for i, (src, defs) in enumerate(UNITS):
            objs.append(os.path.join(obj, f"{i}.o"))
            cmd = [HIPCC] + FLAGS + defs + ["-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c",
                                            os.path.join(CSRC, src), "-o", objs[-1]]
            if verbose:
                print(" ".join(cmd), flush=True)
            jobs.append(subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))
        outs = [j.communicate()[0] for j in jobs]
        if not any(j.returncode for j in jobs):
            res = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-o", tmp] + objs,
                                 capture_output=True, text=True)
            outs.append(res.stdout + res.stderr)
            jobs.append(res)
        if any(j.returncode for j in jobs):
            sys.stderr.write("".join(outs))
            raise RuntimeError("hipcc failed building libpsatd.so")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build()
