"""Build the HIP library libptycho.so in-tree for gfx950.

Run as ``python -m paper_2205_06327_amd.build``; __graft_entry__.build() calls
``build()``.  Every kernel and the C ABI are compiled by hipcc into one shared
object next to this file.
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libptycho.so")
SOURCES = [
    os.path.join(HERE, "csrc", "ptycho_kernels.hip"),
    os.path.join(HERE, "csrc", "tile_kernels.hip"),
    os.path.join(HERE, "csrc", "ptycho_api.cpp"),
    os.path.join(HERE, "csrc", "ptycho_static.hip"),
]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3",
    "--offload-arch=gfx950",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-munsafe-fp-atomics",
    # no packed FP32 instructions anywhere in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]


def build(verbose: bool = False) -> str:
    tmp = LIB + ".tmp"
    cmd = [HIPCC, *FLAGS, *SOURCES, "-o", tmp]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed building libptycho.so")
    if verbose:
        sys.stderr.write(res.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
