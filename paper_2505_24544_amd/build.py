"""Build libbeagle_xattn.so in-tree with hipcc for gfx950.

Usage: python -m paper_2505_24544_amd.build   (or build() from Python).
Every source is recompiled on every call; objects go to csrc/_build/.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libbeagle_xattn.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option",
]
# Matrix instructions write either register file.  By default all of a kernel's write accumulation registers as soon as it needs any
# of those, and every score, probability or sum that vector instructions go on to use is copied over first.  By file, us without / with:
# dK/dV see attn_bwd_bf16.hip; draft step of 64 queries over 4096 rows 57.6 / 56.8, of 16 over 1024 28.8 / 28.5, on packed weights of 12 over
# 3000 in 8 groups 28.5 / 27.8 (the kernels of up to 16 rows take 80 accumulation registers without, none with).  The other
# files' kernels come out the same either way.
VGPR_FORM = ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]
VGPR_FORM_SOURCES = ("attn_bwd_bf16.hip", "decode_bf16.hip")


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src: str) -> str:
    bdir = os.path.join(CSRC, "_build")
    os.makedirs(bdir, exist_ok=True)
    obj = os.path.join(bdir, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, *(VGPR_FORM if src in VGPR_FORM_SOURCES else ()), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
    noise = "packed-fp32-ops' is not a recognized feature"
    warn = "\n".join(l for l in r.stderr.splitlines() if l.strip() and noise not in l)
    if warn.strip():
        sys.stderr.write(warn + "\n")
    return obj


def build(verbose: bool = True) -> str:
    srcs = sources()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", *objs, "-o", OUT]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    if verbose:
        print("built", OUT, "from", ", ".join(srcs))
    return OUT


if __name__ == "__main__":
    build()
