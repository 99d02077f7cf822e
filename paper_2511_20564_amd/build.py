"""Builds libe2eg.so (HIP kernels + C ABI) for gfx950 with hipcc, and the extension _native.so that calls it
from Python with g++, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libe2eg.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["status.hip", "scan.hip", "sort.hip", "build_csr.hip", "normalize.hip", "propagate.hip", "transform.hip", "readout.hip", "sampler.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def needs_build() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(NATIVE):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(NATIVE))
    deps = sources() + [os.path.join(CSRC, f) for f in ("common.h", "radix.h", "entry_tiles.h", "native.cpp")]
    deps.append(os.path.join(HERE, "..", "include", "e2eg.h"))
    return any(os.path.getmtime(d) > t for d in deps)


def build(verbose: bool = True) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    lib = [hipcc] + HIPCC_FLAGS + ["-o", LIB] + sources()
    native = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
              "-I" + sysconfig.get_paths()["include"], "-o", NATIVE, os.path.join(CSRC, "native.cpp"),
              "-L" + HERE, "-l:libe2eg.so", "-Wl,-rpath,$ORIGIN"]
    for cmd in (lib, native):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
