"""Build libexemcl.so in-tree with hipcc for gfx950.

Every translation unit is compiled with packed-fp32 instruction generation
switched off (``-Xclang -target-feature -Xclang -packed-fp32-ops``); hipcc's
host pass warns that it does not know that feature, which is harmless.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OBJDIR = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libexemcl.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

SOURCES = ["host.cpp", "kernels_mfma.hip", "kernels_mfma_f32.hip", "kernels_mfma_f16.hip",
           "kernels_mfma_bf16.hip", "kernels_mfma_split.hip", "kernels_mfma_split_gain.hip",
           "kernels_mfma_split_gather.hip", "kernels_mfma_split_gain_gather.hip", "kernels_mfma_split_rowmax.hip",
           "kernels_mfma_wide.hip", "kernels_mfma_bigd.hip", "kernels_aux.hip", "kernels_greedy.hip",
           "kernels_sqnorm.hip"]
FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-result", f"-I{INCLUDE}", f"-I{CSRC}"]


# The matrix-core kernels: accumulators in VGPRs (the epilogue reads them
# directly), and max without NaN canonicalisation (inputs are finite).
MFMA_FLAGS = ["-mllvm", "-amdgpu-mfma-vgpr-form", "-fno-honor-nans"]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(OBJDIR, os.path.splitext(src)[0] + ".o")
    extra = MFMA_FLAGS if src.startswith("kernels_mfma_") else []
    cmd = [HIPCC, *FLAGS, *extra, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed on {src}")
    noise = "is not a recognized feature for this target"
    msgs = [ln for ln in (r.stdout + r.stderr).splitlines() if ln.strip() and noise not in ln]
    if msgs and verbose:
        print("\n".join(msgs))
    return obj


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compile every source and link the shared library; return its path."""
    os.makedirs(OBJDIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    tmp = f"{LIB}.tmp{os.getpid()}"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
