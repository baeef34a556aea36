"""Builds libnetmax.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libnetmax.so")

SOURCES = ["netmax_api.hip", "k_small_iter.hip", "k_sliced_iter.hip", "k_resident_mlp.hip", "k_sample.hip", "k_synth_grad.hip", "k_mix.hip", "k_consensus.hip", "k_grad_mlp.hip",
           "k_layout.hip", "k_grad_mfma.hip", "k_grad_head.hip", "k_grad_f32.hip", "policy.hip", "k_async.hip", "k_mix_subset.hip", "k_mix_synth.hip",
           "k_tile_fwd.hip", "k_tile_dgrad.hip", "k_tile_wgrad.hip", "k_chain.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-result",
         # packed fp32 instructions are kept out of the generated code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    subprocess.run([HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj], check=True)
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], check=True)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
