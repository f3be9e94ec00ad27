"""Compile in-tree: csrc/zvc.hip -> paper_1705_01626_amd/libzvc.so (the HIP library) and
csrc/calls.cpp -> paper_1705_01626_amd/_calls.so (its entry from Python).

Usage: python -m paper_1705_01626_amd.build
hipcc cross-compiles for gfx950, so this works on a machine without a GPU.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SOURCE = os.path.join(PKG, "csrc", "zvc.hip")
LIBRARY = os.path.join(PKG, "libzvc.so")
CALLS_SOURCE = os.path.join(PKG, "csrc", "calls.cpp")
CALLS = os.path.join(PKG, "_calls.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

ROCM_INCLUDE = os.environ.get("ROCM_INCLUDE", "/opt/rocm/include")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
]


def build(output: str = LIBRARY, extra=()) -> str:
    cmd = [HIPCC, *FLAGS, *extra, "-I", os.path.join(ROOT, "include"), "-o", output, SOURCE]
    subprocess.run(cmd, check=True)
    return output


def build_calls(output: str = CALLS) -> str:
    """The Python entry: host code only; it takes the functions from the loaded library."""
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I", ROCM_INCLUDE,
                    "-I", sysconfig.get_paths()["include"], CALLS_SOURCE, "-o", output, "-ldl"], check=True)
    return output


def ensure_built() -> str:
    """Build only if nothing is built yet (or the source is newer)."""
    if (not os.path.exists(LIBRARY)
            or os.path.getmtime(LIBRARY) < os.path.getmtime(SOURCE)):
        build()
    if (not os.path.exists(CALLS)
            or os.path.getmtime(CALLS) < os.path.getmtime(CALLS_SOURCE)):
        build_calls()
    return LIBRARY


if __name__ == "__main__":
    print(build(extra=sys.argv[1:]))
    print(build_calls())
