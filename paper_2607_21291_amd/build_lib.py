"""Build libadadsf.so (HIP, gfx950) in-tree with hipcc.

Usage: python -m paper_2607_21291_amd.build_lib [-v]
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build", "adadsf")
LIB = os.path.join(PKG, "libadadsf.so")

SOURCES = ["api.hip", "kernels_misc.hip", "kernels_router.hip", "kernels_align.hip", "kernels_gemm.hip",
           "kernels_rowgemm.hip", "kernels_attn.hip", "kernels_decode.hip", "kernels_wgrad.hip", "kernels_bwd.hip"]
# per-source extra flags: attention keeps its MFMA accumulators in ordinary
# VGPRs, so the softmax reads scores and rescales outputs without AGPR moves
EXTRA = {"kernels_attn.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
         "kernels_gemm.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
         "kernels_rowgemm.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
         "kernels_decode.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
         "kernels_wgrad.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
         "kernels_bwd.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}

ARCH = "gfx950"
CFLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # keep every fp32 operation scalar: no packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
    "-I", INCLUDE, "-I", CSRC,
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build libadadsf.so)")


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(line for line in (res.stdout + res.stderr).splitlines()
                     if "packed-fp32-ops" not in line)  # host pass does not know the feature
    if res.returncode != 0:
        raise RuntimeError(f"command failed ({res.returncode}): {' '.join(cmd)}\n{out}")
    if verbose and out.strip():
        print(out)


def build(verbose: bool = False) -> str:
    """Compile every source for gfx950 and link libadadsf.so next to this file."""
    os.makedirs(BUILD, exist_ok=True)
    cc = hipcc()
    objs = []
    jobs = []
    with cf.ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 4)) as ex:
        for src in SOURCES:
            obj = os.path.join(BUILD, src.replace(".hip", ".o"))
            objs.append(obj)
            cmd = [cc, *CFLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
            jobs.append(ex.submit(_run, cmd, verbose))
        for j in jobs:
            j.result()
    tmp = LIB + ".tmp"
    _run([cc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
