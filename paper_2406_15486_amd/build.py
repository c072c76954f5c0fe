"""Build the HIP library in-tree with hipcc for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsampleattn.so")
SOURCES = ["sa_api.hip", "flash_attn.hip", "prep.hip", "scores.hip", "select.hip", "probes.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-munsafe-fp-atomics",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument", "-Wno-inline-asm",
]
# flash_attn.hip: wave-uniform branches stay branches.  The structurizer otherwise turns the uniform if / else of the
# tile loops into flag chains, whose joins hold every array twice (90 to 270 bytes of spills per lane;
# tests/test_build.py looks for them, should a compiler drop the option).
EXTRA_FLAGS = {"flash_attn.hip": ["-mllvm", "-structurizecfg-skip-uniform-regions=1"]}


def build(verbose: bool = True, extra: list[str] | None = None) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

    def run(cmd: list[str]) -> None:
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)

    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(len(SOURCES)) as pool:
        objects = [os.path.join(tmp, s + ".o") for s in SOURCES]
        list(pool.map(run, [[hipcc, "-c", *FLAGS, *EXTRA_FLAGS.get(s, []), *(extra or []), os.path.join(CSRC, s), "-o", o]
                            for s, o in zip(SOURCES, objects)]))
        run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objects, "-o", LIB])
    return LIB


if __name__ == "__main__":
    build(extra=sys.argv[1:])
