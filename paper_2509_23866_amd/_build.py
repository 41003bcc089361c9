"""Build step for libdart.so (hipcc, gfx950) and the binding's native marshalling
(the host compiler, against torch). Always compiles when called."""

from __future__ import annotations

import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRCS = [os.path.join(HERE, "csrc", n) for n in ("dart.hip", "lmhead.hip", "check.hip")]
LIB = os.path.join(HERE, "libdart.so")
NATIVE_SRC = os.path.join(HERE, "csrc", "binding.cpp")
NATIVE = os.path.join(HERE, "_native.so")
INCLUDE = os.path.join(ROOT, "include")

HIPCC_FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-shared", "-Werror=shadow",
    # packed-FP32 VALU forms stay disabled: plain scalar fp32 code only
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def build(verbose: bool = False, extra_flags=(), out: str = LIB) -> str:
    cmd = ["hipcc", *HIPCC_FLAGS, *extra_flags, "-I", INCLUDE, *SRCS, "-o", out]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return out


def build_native(verbose: bool = False, out: str = NATIVE) -> str:
    """_native.so: host code only (CPython and torch's C++ API; libdart.so is
    opened at run time)."""
    import torch

    base = os.path.dirname(torch.__file__)
    system = [os.path.join(base, "include"),
              os.path.join(base, "include", "torch", "csrc", "api", "include"),
              os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"),
              sysconfig.get_paths()["include"]]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           # what torch's and HIP's headers are written against here
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", INCLUDE,
           *[x for d in system for x in ("-isystem", d)], NATIVE_SRC, "-o", out,
           "-L", os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return out


if __name__ == "__main__":
    build(verbose=True)
    build_native(verbose=True)
