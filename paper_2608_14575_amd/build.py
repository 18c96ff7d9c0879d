"""Build libhwr.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2608_14575_amd.build
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
LIB = os.path.join(PKG, "libhwr.so")
BUILD = os.path.join(PKG, "_build")

SOURCES = ["hwr_api.hip", "k_common.hip", "k_bf16.hip", "k_table.hip", "k_route.hip", "k_f32.hip",
           "k_single.hip", "k_probe.hip", "hwr_sim.cpp"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # no packed-fp32 instructions in device code; no multiply-add contraction:
    # every fp32 operation of the decision is rounded once, as documented (fused
    # multiply-adds are written as fmaf where they are meant)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-ffp-contract=off",
    "-Wall", "-Wno-unused-function",
    f"-I{INCLUDE}", f"-I{CSRC}",
]


# Per-source flags.  MFMA results in vector registers (VGPR form): k_bf16.hip,
# so that the accumulation registers stay free for the four-tile predictor's
# first-layer activations, which its MFMAs read directly; k_table.hip,
# k_route.hip and k_f32.hip, whose vector code reads the results.
EXTRA = {k: ["-mllvm", "-amdgpu-mfma-vgpr-form"] for k in ("k_bf16.hip", "k_table.hip", "k_route.hip", "k_f32.hip")}


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    """Compile every source and link libhwr.so (always rebuilds)."""
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
