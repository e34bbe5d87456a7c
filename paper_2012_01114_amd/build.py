"""Build libattnring.so (HIP, gfx950 only) in-tree.

`python -m paper_2012_01114_amd.build` or `build()`; objects go to
paper_2012_01114_amd/_build/, the library next to this file.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libattnring.so")
PROBE_LIB = os.path.join(HERE, "libattnprobe.so")   # ceilings probe: instrumentation, its own library
SOURCES = ["attnring_api.hip", "generic_kernels.hip", "proj_split.hip", "attn_float.hip", "attn_planes.hip", "proj_attn_small.hip",
           "proj_mfma.hip", "attn_pipe.hip", "attn_split.hip", "attn_strands.hip",
           "sym_pair.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# Loops start on a 64-byte line (the kernels that walk through LDS): where the walk of attn_pipe_kernel<128, FULL> happened to start was worth 4 to 7 %
# (one item of 4096 vectors, 4 heads: 94.8 -> 88.3 us, at the same instructions).  In the GEMMs it costs more than it
# gives (960 x 1456 -> 1536: 20.7 -> 21.4).
FLAGS_OF = {"attn_pipe.hip": ["-falign-loops=64"], "attn_strands.hip": ["-falign-loops=64"]}


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + FLAGS + FLAGS_OF.get(src, []) + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(_compile, SOURCES + ["ceilings_probe.hip"]))
    for lib, members in ((LIB, objs[:-1]), (PROBE_LIB, objs[-1:])):
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib] + members
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
