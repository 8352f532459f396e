"""Build libsparseloco.so (hipcc, gfx950) and _calls.so, the binding's way into it, next to this file.

    python -m paper_2601_02360_amd.build

Both are built in-tree so that they travel with the source tree; they are
git-ignored.  There is no other code path: if the library is missing the
binding raises.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = [os.path.join(HERE, "csrc", name) for name in ("sparseloco.hip", "subspace.hip", "stream_probe.hip")]
LIB = os.path.join(HERE, "libsparseloco.so")
CALLS = os.path.join(HERE, "_calls.so")

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
    "-ffp-contract=off",
    # keep the compiler from forming packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]


def _run(cmd, out: str, verbose: bool) -> None:
    tmp = out + ".tmp%d" % os.getpid()
    cmd = cmd + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, out)


def build(verbose: bool = False, extra=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    _run([hipcc, *HIPCC_FLAGS, *extra, *SOURCES], LIB, verbose)
    build_calls(verbose)
    return LIB


def build_calls(verbose: bool = False) -> str:
    import torch
    at = os.path.dirname(torch.__file__)
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
          "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, os.path.join(HERE, "csrc", "calls.cpp"),
          "-I", os.path.join(ROOT, "include"), "-isystem", os.path.join(at, "include"),
          "-isystem", os.path.join(at, "include", "torch", "csrc", "api", "include"),
          "-isystem", sysconfig.get_paths()["include"], "-isystem", "/opt/rocm/include",
          "-L", HERE, "-lsparseloco", "-L", os.path.join(at, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10",
          "-Wl,-rpath,$ORIGIN"], CALLS, verbose)
    return CALLS


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
    print("built", LIB)
