"""Builds libhgnn.so (HIP, gfx950 only) in-tree with hipcc, and with g++ the module that calls it from torch tensors."""
from __future__ import annotations

import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libhgnn.so")
CALLS_PATH = os.path.join(HERE, "_calls.so")
SOURCES = ["memory.hip", "plan.hip", "tasks.hip", "blocked.hip", "groups.hip", "spmm.hip", "spmm_static.hip", "slices.hip", "sddmm.hip", "gat.hip", "gat_bwd.hip", "softmax.hip", "transpose.hip", "dense.hip"]
# packed-fp32 instructions are switched off on purpose (the compiler must not emit v_pk_*_f32)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def compile_calls(source: str, out: str, flags=(), verbose: bool = False) -> None:
    """Compile host code that takes torch tensors and Python arguments."""
    import torch

    base = os.path.dirname(torch.__file__)
    # NDEBUG: else the headers bring a thread-local counter along, and behind a library with thread-local memory that is loaded late and never uses it
    # every access to such memory in the runtime takes glibc's slow way (2 us more for a set-up call)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-DNDEBUG", "-std=c++17", "-shared", "-fPIC", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", os.path.join(base, "include"), "-I", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"),
           *flags, source, "-o", out, "-L", os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)


def build_calls(verbose: bool = False) -> str:
    """Compile csrc/calls.cpp (Python arguments to the library's entry points)."""
    compile_calls(os.path.join(CSRC, "calls.cpp"), CALLS_PATH, verbose=verbose)
    return CALLS_PATH


def build(verbose: bool = False) -> str:
    """Compile every translation unit and link the shared library; always recompiles."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)

    def one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        return obj

    with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1)) as ex:
        objs = list(ex.map(one, SOURCES))
    build_calls(verbose)
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs, "-L/opt/rocm/lib", "-lhsa-runtime64"])
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
