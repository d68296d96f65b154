"""Build libgenerals.so for gfx950 with hipcc (in-tree, no JIT cache).

    python -m paper_2606_23348_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgenerals.so")
SOURCES = ["kernels.hip", "features.hip", "transfer.hip", "abi.cpp", "server.cpp"]
ARCH = os.environ.get("GEN_OFFLOAD_ARCH", "gfx950")

HIPCC_FLAGS = [
    "-x", "hip", f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-Wall", "-Wno-unused-function",
    # no packed fp32 instructions anywhere in this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def build(verbose: bool = False, extra: list | None = None) -> str:
    """Compile the sources side by side, link them, put the library in place."""
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    with tempfile.TemporaryDirectory(prefix="gen_build_") as d:
        objs = [os.path.join(d, s + ".o") for s in SOURCES]

        def compile_one(i: int) -> None:
            cmd = [hipcc, *HIPCC_FLAGS, *(extra or []), "-c", "-o", objs[i], os.path.join(CSRC, SOURCES[i])]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.check_call(cmd)

        with ThreadPoolExecutor(len(SOURCES)) as ex:
            list(ex.map(compile_one, range(len(SOURCES))))
        tmp = LIB + ".tmp%d" % os.getpid()
        subprocess.check_call([hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
    print(LIB)
