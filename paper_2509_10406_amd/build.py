"""Builds libmuse.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmuse.so")
SOURCES = ["muse_api.hip", "kmeans.hip", "attn_simple.hip", "attn_fp32.hip", "attn_fwd.hip", "attn_bwd.hip", "attn_mfma.hip", "farfield.hip", "farfield_tiles.hip", "farfield_bwd.hip", "cell_grads.hip", "chain_grads.hip", "retrieval.hip", "retrieval_fp32.hip", "retrieval_kv.hip", "retrieval_q.hip", "dipole.hip", "probe.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# attn_bwd.hip: matrix instructions write vector registers; what stays in accumulation registers is said there
FILE_FLAGS = {"attn_bwd.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}


def build(verbose: bool = False) -> str:
    objs = []
    procs = []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    for s in SOURCES:
        o = os.path.join(HERE, "_build", s.replace(".hip", ".o"))
        objs.append(o)
        procs.append((s, subprocess.Popen(["hipcc", *FLAGS, *FILE_FLAGS.get(s, []), "-c", os.path.join(CSRC, s), "-o", o],
                                          stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for s, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {s}:\n{out}")
        if verbose and out.strip():
            print(out)
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
