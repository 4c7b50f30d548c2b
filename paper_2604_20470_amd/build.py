"""Compile the gfx950 library in-tree with hipcc: paper_2604_20470_amd/libdynamicrad.so."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdynamicrad.so")
SOURCES = ["dr_api.hip", "k_scores.hip", "k_mask.hip", "k_attn_split.hip", "k_attn_mfma.hip", "k_attn_mfma_small.hip", "k_attn_mfma_pair.hip", "k_attn_mfma_duo.hip", "k_tokens.hip", "k_proxy.hip", "k_clock_probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 instructions
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
    "-Wno-inline-asm",          # m0 is named as clobbered by the tile-load asm; clang warns that it is a reserved register
]


def build(verbose: bool = False, force: bool = True) -> str:
    """Compile every source and link the shared library.  Returns the library path."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    headers = [os.path.join(CSRC, "dr_internal.h"), os.path.join(CSRC, "attn_mfma_common.h"), os.path.join(CSRC, "attn_pair_body.h"), os.path.join(HERE, "..", "include", "dynamicrad.h"),
               os.path.join(HERE, "..", "include", "dynamicrad_probe.h")]
    hdr_time = max(os.path.getmtime(h) for h in headers)

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        path = os.path.join(CSRC, src)
        if not force and os.path.exists(obj) and os.path.getmtime(obj) > max(os.path.getmtime(path), hdr_time):
            return obj
        cmd = [HIPCC, *FLAGS, "-c", path, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
        if verbose and r.stderr.strip():
            print(r.stderr, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", *objs, "-o", LIB]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, force="--incremental" not in sys.argv))
