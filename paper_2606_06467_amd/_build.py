"""Build libclsa.so (gfx950 only) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libclsa.so")
BUILD_DIR = os.path.join(PKG, "_build")

SOURCES = ["index_decode.hip", "index_prefill.hip", "topk.hip", "sparse_attn.hip", "tile_attn.hip",
           "project.hip", "kd.hip", "kd_loss.hip", "noalloc.hip",
           "api.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

COMMON_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-fPIC", "-std=c++17", "-Wall",
    # no packed fp32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", INCLUDE, "-I", CSRC,
]


# Per-source flags: matrix-core results in ordinary VGPRs.  kd.hip: no
# accumulator-register copies before the exponentials that consume them;
# sparse_attn.hip: the chunked-prefill form of the layer kernel fits four waves
# per SIMD; tile_attn.hip: the logits and the rescaled accumulators feed vector
# instructions.  kd_loss.hip goes without: its 128 gradient accumulators are
# touched by matrix instructions only and fit beside the rest as accumulator
# registers (3.2 ms; 4.3 ms in VGPRs).
SOURCE_FLAGS = {"kd.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
                "sparse_attn.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
                "tile_attn.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *COMMON_FLAGS, *SOURCE_FLAGS.get(src, []), "-x", "hip", "-c",
           os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    """Compile every source for gfx950 and link ``libclsa.so``; returns its path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    with ThreadPoolExecutor(len(SOURCES)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
