"""Compiles the HIP library libs2dw.so for gfx950 in-tree (hipcc, no JIT cache)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libs2dw.so")
BUILD = os.path.join(HERE, "_build")

SOURCES = ["persist.hip", "api.cpp", "tables.cpp", "wigner.hip", "stages.hip", "misc.hip"]
# sources compiled apart, for time, and joined into the object of the first
JOINED = {"stages.hip": ["fused_fwd.hip", "fused_adj.hip", "fused_fwd_cx.hip", "fused_adj_cx.hip", "fused_blk.hip"]}

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = os.environ.get("S2DW_ARCH", "gfx950")
FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
         # packed FP32 instructions are kept out of every kernel
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(HERE, "..", "include"), "-I", CSRC]


def _object(src: str) -> str:
    return os.path.join(BUILD, os.path.splitext(src)[0] + ".o")


def _compile(src: str) -> str:
    obj = _object(src) + (".part" if src in JOINED else "")
    cmd = [HIPCC, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj] + FLAGS
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed on {src}")
    return obj


def _join(src: str, parts: list[str]) -> None:
    r = subprocess.run(["ld", "-r", "-o", _object(src)] + parts, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"ld -r failed for {src}")


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as ex:
        every = SOURCES + [p for parts in JOINED.values() for p in parts]
        made = dict(zip(every, ex.map(_compile, every)))
    for src, parts in JOINED.items():
        _join(src, [made[src]] + [made[p] for p in parts])
    objs = [_object(s) for s in SOURCES]
    tmp = OUT + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("link failed")
    os.replace(tmp, OUT)
    if verbose:
        print("built", OUT)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
