"""Build the HEOM library (libheom.so) in-tree for gfx950 with hipcc."""

from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libheom.so")
SOURCES = [os.path.join(CSRC, f) for f in ("heom_kernels.hip", "heom_packed.hip", "heom_columns.hip", "heom_resident.hip", "heom_host.cpp",
                                           "heom_server.cpp", "heom_scratch.hip")]

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    # no packed-FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose=False):
    """Compile every source (side by side) and link the library."""
    with tempfile.TemporaryDirectory() as tmp:
        cmds = []
        for src in SOURCES:
            obj = os.path.join(tmp, os.path.basename(src) + ".o")
            cmds.append([hipcc(), *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                         "-c", src, "-o", obj])
        if verbose:
            for cmd in cmds:
                print(" ".join(cmd), flush=True)
        with concurrent.futures.ThreadPoolExecutor(max_workers=4) as pool:
            list(pool.map(lambda cmd: subprocess.run(cmd, check=True), cmds))
        subprocess.run([hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950",
                        *[cmd[-1] for cmd in cmds], "-o", LIB + ".tmp"], check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
