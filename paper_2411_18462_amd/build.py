"""Builds libsvip.so (HIP kernels + C ABI) for gfx950 with hipcc, and the binding's host module with g++, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = [os.path.join(HERE, "csrc", "svip_kernels.hip"), os.path.join(HERE, "csrc", "svip_loop.hip")]
HEADERS = sorted(os.path.join(HERE, "csrc", f) for f in os.listdir(os.path.join(HERE, "csrc")) if f.endswith(".h")) + \
    [os.path.join(ROOT, "include", "svip.h")]
LIB = os.path.join(HERE, "libsvip.so")
MARSHAL_SRC = os.path.join(HERE, "csrc", "marshal.cpp")
MARSHAL = os.path.join(HERE, "_marshal.so")
EXAMPLE_SRC = os.path.join(HERE, "examples", "round_from_file.cpp")
EXAMPLE_BIN = os.path.join(HERE, "examples", "round_from_file")

# packed-fp32 instructions are switched off for all device code of this library
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-shared", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"),
]


def build(verbose: bool = False) -> str:
    """Compile every HIP source of the package; returns the library path."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + f".tmp{os.getpid()}"
    cmd = [hipcc, *HIPCC_FLAGS, *SOURCES, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in proc.stdout.splitlines()
                    if "is not a recognized feature for this target" not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    os.replace(tmp, LIB)
    build_marshal(verbose)
    build_example(verbose)
    return LIB


def build_marshal(verbose: bool = False) -> str:
    """The binding's native argument marshalling: host code only, against the headers of the torch that is imported."""
    import torch

    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    tmp = MARSHAL + f".tmp{os.getpid()}"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1",
           "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I" + sysconfig.get_paths()["include"],
           "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include", MARSHAL_SRC,
           "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10", "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode != 0:
        raise RuntimeError("g++ failed on the marshalling module:\n" + proc.stdout)
    os.replace(tmp, MARSHAL)
    return MARSHAL


def build_example(verbose: bool = False) -> str:
    """The C-ABI example program (plain HIP host code linked against libsvip.so, found at run time
    through an rpath relative to the executable)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = EXAMPLE_BIN + f".tmp{os.getpid()}"
    cmd = [hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "include"), EXAMPLE_SRC,
           "-L" + HERE, "-lsvip", "-Wl,-rpath,$ORIGIN/..", "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed on the example:\n" + proc.stdout)
    os.replace(tmp, EXAMPLE_BIN)
    return EXAMPLE_BIN


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    if not os.path.exists(EXAMPLE_BIN) or not os.path.exists(MARSHAL):
        return True
    return any(os.path.getmtime(p) > t for p in SOURCES + HEADERS + [EXAMPLE_SRC, MARSHAL_SRC])


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
