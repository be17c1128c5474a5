"""Compile the HIP library for gfx950 in-tree (hipcc cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblonglive.so")
SOURCES = ["api.cpp", "api_prompt.cpp", "api_clip.cpp", "api_diag.cpp", "cache_index.cpp", "append_kernel.hip", "out_proj.hip", "attn_kernel.hip", "attn_stream.hip", "attn_stream16.hip", "attn_resident.hip", "probe_kernels.hip",
           "append_fp8.hip", "attn_fp8.hip", "attn_bwd.hip", "clip_layout.hip"]
# Packed-fp32 VALU forms are switched off for every device translation unit.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def build(verbose: bool = False) -> str:
    """Compile every source into liblonglive.so; raises on failure.  Returns the path."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *FLAGS, *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB + ".tmp"]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in proc.stderr.splitlines() if "packed-fp32-ops' is not a recognized feature" not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + " ".join(cmd) + "\n" + err)
    os.replace(LIB + ".tmp", LIB)
    if verbose and err.strip():
        print(err)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
