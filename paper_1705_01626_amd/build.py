"""Compile in-tree: csrc/zvc.hip -> paper_1705_01626_amd/libzvc.so (the HIP library) and
csrc/calls.cpp -> paper_1705_01626_amd/_calls.<interpreter's tag>.so (its entry from Python,
which is left out where the interpreter's headers are not installed).

Usage: python -m paper_1705_01626_amd.build
hipcc cross-compiles for gfx950, so this works on a machine without a GPU.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from typing import Optional

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SOURCE = os.path.join(PKG, "csrc", "zvc.hip")
LIBRARY = os.path.join(PKG, "libzvc.so")
CALLS_SOURCE = os.path.join(PKG, "csrc", "calls.cpp")
HEADER = os.path.join(ROOT, "include", "zvc.h")
CALLS = os.path.join(PKG, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))   # no other interpreter loads it
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ROCM_INCLUDE = os.environ.get("ROCM_INCLUDE", os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include"))

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


def build_calls(output: str = CALLS) -> Optional[str]:
    """The Python entry: host code only; it takes the functions from the loaded library.  None, with a
    line that says so, if the interpreter's headers are not there: the calls then go through ctypes."""
    include = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(include, "Python.h")):
        print("_calls is not built: no Python.h in %s; device calls go through ctypes" % include, file=sys.stderr)
        return None
    subprocess.run([HIPCC, "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-no-hip-rt", "-Wall", "-Wextra",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I", ROCM_INCLUDE,
                    "-I", include, CALLS_SOURCE, "-o", output, "-ldl"], check=True)
    return output


def _older(output: str, *sources: str) -> bool:
    return not os.path.exists(output) or any(os.path.getmtime(output) < os.path.getmtime(s) for s in sources)


def ensure_built() -> str:
    """Build only what is not built yet (or whose sources are newer)."""
    if _older(LIBRARY, SOURCE, HEADER):
        build()
    if _older(CALLS, CALLS_SOURCE, HEADER):
        build_calls()
    return LIBRARY


if __name__ == "__main__":
    print(build(extra=sys.argv[1:]))
    print(build_calls())
