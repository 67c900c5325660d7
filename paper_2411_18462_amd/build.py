"""Builds libsvip.so (HIP kernels + C ABI) for gfx950 with hipcc, and the binding's host module with g++, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = [os.path.join(HERE, "csrc", "svip_kernels.hip"), os.path.join(HERE, "csrc", "svip_loop.hip")]
ABI = os.path.join(ROOT, "include", "svip.h")
HEADERS = sorted(os.path.join(HERE, "csrc", f) for f in os.listdir(os.path.join(HERE, "csrc")) if f.endswith(".h")) + [ABI]
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


def _compile(cmd: list[str], out: str, verbose: bool) -> str:
    """Runs a compiler command whose output goes to a temporary file beside `out`; returns that file's name."""
    tmp = out + f".tmp{os.getpid()}"
    cmd = [*cmd, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        said = "\n".join(l for l in proc.stdout.splitlines() if "is not a recognized feature for this target" not in l)
        if proc.returncode != 0:
            raise RuntimeError(f"{os.path.basename(cmd[0])} failed on {os.path.basename(out)}:\n{said}")
    except BaseException:
        if os.path.exists(tmp):
            os.remove(tmp)
        raise
    if verbose and said.strip():
        print(said)
    return tmp


def build(verbose: bool = False) -> str:
    """Compile every source of the package; returns the library path.  The library and the binding's module, which calls it by
    address, take their places together, once both have been compiled."""
    lib = _compile([_hipcc(), *HIPCC_FLAGS, *SOURCES], LIB, verbose)
    try:
        marshal = _compile(_marshal_command(), MARSHAL, verbose)
    except BaseException:
        os.remove(lib)
        raise
    os.replace(lib, LIB)
    os.replace(marshal, MARSHAL)
    build_example(verbose)
    return LIB


def _hipcc() -> str:
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _marshal_command() -> list[str]:
    """The binding's native argument marshalling: host code only, against the headers of the torch that is imported."""
    import torch

    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1",
            "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I" + sysconfig.get_paths()["include"],
            "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include", MARSHAL_SRC,
            "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]


def build_example(verbose: bool = False) -> str:
    """The C-ABI example program (plain HIP host code linked against libsvip.so, found at run time
    through an rpath relative to the executable)."""
    os.replace(_compile([_hipcc(), "--offload-arch=gfx950", "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "include"), EXAMPLE_SRC,
                         "-L" + HERE, "-lsvip", "-Wl,-rpath,$ORIGIN/.."], EXAMPLE_BIN, verbose), EXAMPLE_BIN)
    return EXAMPLE_BIN


def is_stale() -> bool:
    """Whether something that build() makes is missing or older than what it is made from."""
    products = ((LIB, SOURCES + HEADERS), (MARSHAL, [MARSHAL_SRC, ABI]), (EXAMPLE_BIN, [EXAMPLE_SRC, ABI]))
    return any(not os.path.exists(out) or any(os.path.getmtime(p) > os.path.getmtime(out) for p in made_from)
               for out, made_from in products)


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
