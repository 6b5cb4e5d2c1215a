"""Builds liballocmoe.so (hand-written HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liballocmoe.so")
# (the four that take a minute each come first)
SOURCES = ["ffn_bf16_t256_ffn1.hip", "ffn_bf16_t256_ffn2.hip", "ffn_bf16_t256_ffn1_fp8.hip",
           "ffn_bf16_t256_ffn2_fp8.hip", "api.hip", "route.hip", "plan.hip", "pack.hip",
           "ffn_f32.hip", "ffn_bf16.hip", "ffn_bf16_t256.hip", "combine.hip",
           "stats.hip", "probes.hip", "alloc_l.cpp"]
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-Wall", "-Wno-inline-asm", "-Wno-unused-command-line-argument", "-Wno-unknown-attributes"]


def build_library(verbose: bool = False, jobs: int = 8) -> str:
    """Compile every kernel source and link the shared library.  Always compiles."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs, objs = [], []
    for src in SOURCES:
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        objs.append(obj)
        cmd = [hipcc, *HIPCC_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
        if len(procs) >= jobs:
            _drain(procs)
    _drain(procs)
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.check_call(cmd)
    return LIB


def _drain(procs):
    while procs:
        src, p = procs.pop(0)
        out, _ = p.communicate()
        text = out.decode(errors="replace")
        # hipcc's host pass does not know the packed-fp32 target feature: harmless
        lines = [l for l in text.splitlines() if "packed-fp32-ops" not in l and l.strip()]
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{text}")
        if lines:
            print(f"[{src}]\n" + "\n".join(lines), flush=True)


if __name__ == "__main__":
    print(build_library(verbose=True))
