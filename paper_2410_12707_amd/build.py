"""Builds libadatopk.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree, and next to it
libadatopk_measure.so: the same sources compiled with ADATOPK_MEASURE_BUILD, which adds the
benchmark-only hooks of include/adatopk_measure.h (per-kernel dispatch timing, plain streaming
kernels).  The product library carries none of them.  _marshal is the Python extension that reads
the arguments and makes the calls (marshal.cpp, host code only); the package works without it."""
from __future__ import annotations

import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libadatopk.so")
MEASURE_LIB = os.path.join(HERE, "libadatopk_measure.so")
# (the suffix names the Python it is built for: another one does not load it)
MARSHAL_LIB = os.path.join(HERE, "_marshal" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
MARSHAL_SOURCE = os.path.join(CSRC, "marshal.cpp")
HEADER = os.path.join(ROOT, "include", "adatopk.h")
SOURCES = [os.path.join(CSRC, "adatopk.hip"), os.path.join(CSRC, "adatopk_host.cpp")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
    # packed-fp32 instruction forms are kept out of the generated code on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def build_library(verbose: bool = False, out: str = LIB, defines=()) -> str:
    """Compiles the library to `out`; `defines` are extra -D macros (launch-shape overrides)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + HIPCC_FLAGS + ["-D" + d for d in defines] + ["-o", out] + SOURCES
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return out


def build_measure_library(verbose: bool = False) -> str:
    return build_library(verbose, MEASURE_LIB, ("ADATOPK_MEASURE_BUILD",))


def build_marshal(verbose: bool = False) -> str:
    """The Python extension that reads the arguments and makes the calls (host code only)."""
    import torch

    base = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-isystem", os.path.join(base, "include"), "-isystem", os.path.join(base, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"), "-Wall", "-Wextra", "-o", MARSHAL_LIB, MARSHAL_SOURCE,
           "-L" + os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return MARSHAL_LIB


def library_is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = SOURCES + [HEADER, os.path.join(ROOT, "include", "adatopk_measure.h"), os.path.join(CSRC, "wire_layout.h")]
    return any(os.path.getmtime(d) > t for d in deps)


def marshal_is_stale() -> bool:
    if not os.path.exists(MARSHAL_LIB):
        return True
    t = os.path.getmtime(MARSHAL_LIB)
    return any(os.path.getmtime(d) > t for d in (MARSHAL_SOURCE, HEADER))  # (it calls the library's functions by address, as the header declares them)


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_measure_library(verbose=True))
    print(build_marshal(verbose=True))
