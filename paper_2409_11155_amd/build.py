"""Builds libiso.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libiso.so")

SOURCES = ["iso_api.hip", "elementwise.hip", "gemm_simple.hip", "gemm_bf16_mfma.hip", "gemm_bf16_dtl.hip", "gemm_fp8_dtl.hip", "gemm_pp.hip", "gemm_split.hip", "gemm_f32.hip", "attn_f32.hip", "attn_simple.hip",
           "attn_bf16_mfma.hip", "attn_bf16_dtl.hip", "attn_bf16_wave.hip"]


# what decides the device code
DEVICE_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found; libiso cannot be built")


def build(verbose: bool = True) -> str:
    """Compiles every HIP source for gfx950 and links libiso.so next to this file."""
    cmd = [hipcc(), *DEVICE_FLAGS, "-fPIC", "-shared", "-Wno-unused-command-line-argument", "-o", LIB_PATH] + [os.path.join(CSRC, s) for s in SOURCES]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass warns that it does not know the packed-fp32 feature: harmless, drop it
    err = "\n".join(l for l in proc.stderr.splitlines() if "packed-fp32-ops" not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + proc.stdout + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)
    return LIB_PATH


if __name__ == "__main__":
    print(build())
