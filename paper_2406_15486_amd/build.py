"""Build the HIP library in-tree with hipcc for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsampleattn.so")
SOURCES = ["sa_api.hip", "flash_attn.hip", "prep.hip", "scores.hip", "select.hip", "probes.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-munsafe-fp-atomics",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # Wave-uniform branches stay branches: the structurizer otherwise turns the uniform if / else of the tile
    # loops into flag chains, whose joins hold every array twice (360 to 570 bytes of spills per lane).
    "-mllvm", "-structurizecfg-skip-uniform-regions=1",
    "-Wno-unused-command-line-argument", "-Wno-inline-asm",
]


def build(verbose: bool = True, extra: list[str] | None = None) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *FLAGS, *(extra or []), *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    build(extra=sys.argv[1:])
