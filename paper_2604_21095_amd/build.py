"""Build libtgw.so (the gfx950 kernels + C ABI) in this package directory."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libtgw.so")
SOURCES = [os.path.join(HERE, "csrc", f) for f in ("tgw_kernels.hip", "tgw_small.hip", "tgw_runtime.hip", "tgw_bed.hip", "tgw_arena.hip")]
HEADERS = [os.path.join(ROOT, "include", h) for h in ("tgw.h", "tgw_debug.h")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # keep the compiler from emitting packed FP32 VALU instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-unused-function",
    "-pthread",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False) -> str:
    """Compile the HIP library (always recompiles) and check the header as C."""
    tmp = LIB + ".tmp"

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)

    with tempfile.TemporaryDirectory() as d:  # one compiler per source, side by side
        objects = [os.path.join(d, os.path.basename(s) + ".o") for s in SOURCES]
        with ThreadPoolExecutor(len(SOURCES)) as pool:
            list(pool.map(lambda so: run([hipcc(), *HIPCC_FLAGS, "-c", "-I", os.path.join(ROOT, "include"), so[0], "-o",
                                          so[1]]), zip(SOURCES, objects)))
        run([hipcc(), *HIPCC_FLAGS, "-shared", *objects, "-o", tmp])
    os.replace(tmp, LIB)
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc:
        for h in HEADERS:
            subprocess.run([cc, "-std=c99", "-Wall", "-Werror", "-fsyntax-only", "-x", "c", h], check=True)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
    print(LIB)
