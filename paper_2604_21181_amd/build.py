"""Build the mbem HIP library for gfx950 in-tree (libmbem.so next to this file).

    python -m paper_2604_21181_amd.build

Every translation unit is compiled by hipcc for gfx950 only.  Packed FP32
instructions are disabled for the device code (-packed-fp32-ops).
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmbem.so")
BUILD = os.path.join(HERE, "_build")

SOURCES = ["host_mesh.cpp", "capi.cpp", "pool.cpp", "geom.hip", "fill.hip", "pairs.hip", "ssq.hip", "linalg.hip",
           "post.hip", "gemm.hip", "block.hip", "adjoint.hip", "shape.hip", "blr.hip", "near.hip"]
ARCH = os.environ.get("MBEM_OFFLOAD_ARCH", "gfx950")


def hipcc() -> str:
    for c in (os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc"),
              shutil.which("hipcc") or ""):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def _flags(src: str):
    f = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-Wall",
         "-Wno-unused-function", "-Wno-unused-variable"]
    if src.endswith(".hip"):
        f += ["-x", "hip", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
              "-ffp-contract=fast"]
    if src in ("fill.hip", "pairs.hip", "ssq.hip", "shape.hip"):
        # machine-level loop-invariant code motion hoists every constant of
        # the Sauter-Schwab kernels' point loops into registers (248 instead
        # of 222 VGPRs), which measured 10 % slower, and those of the FP64
        # pair kernels into scalar registers that then spill (38, and 168
        # instead of 152 VGPRs); k_shape_regular spills 28 bytes with it
        f += ["-mllvm", "-disable-machine-licm"]
    return f


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    cc = hipcc()

    def compile_one(src):
        obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
        cmd = [cc, *_flags(src), "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
        if verbose and r.stderr.strip():
            print(r.stderr, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=min(6, os.cpu_count() or 1)) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [cc, "-shared", "-fPIC", f"--offload-arch={ARCH}", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
