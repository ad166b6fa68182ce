"""Builds the gfx950 shared library (C ABI of include/rtn.h) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "librtn_gfx950.so")
NATIVE_PATH = os.path.join(PKG_DIR, "_native.so")
SOURCES = ["rtn_api.hip", "rtn_quantize.hip", "rtn_linear.hip", "rtn_linear_wide.hip", "rtn_linear_block4.hip", "rtn_linear_block4z.hip",
           "rtn_linear_block8.hip", "rtn_linear_block8z.hip", "rtn_gemm_tile.hip", "rtn_bench.hip"]
# The block kernel's instantiations are translation units of their own so that they compile side by side (one unit takes minutes).  They
# are joined with the unit that launches them into one object: the host tests link the library's objects by name around a driver of
# their own, and an object that refers to the others would have to be listed with them everywhere.
JOINED = {"rtn_linear_wide.o": ["rtn_linear_wide.o", "rtn_linear_block4.o", "rtn_linear_block4z.o", "rtn_linear_block8.o", "rtn_linear_block8z.o"]}
HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
    # no packed-fp32 instruction selection: some packed fp32 forms have given wrong results on this platform
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def build_native(verbose: bool = False) -> str:
    """Compiles the binding's native calls (host code only) against the installed PyTorch.  The module says what it was compiled for: the
    binding loads it with nothing else."""
    import re
    import sysconfig
    from importlib.util import find_spec
    torch_dir = os.path.dirname(find_spec("torch").origin)
    with open(os.path.join(torch_dir, "version.py")) as f:
        version = re.search(r"__version__ = '([^']+)'", f.read()).group(1)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unused-function", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
           f'-DRTN_BUILT_FOR="torch {version}, Python {sysconfig.get_python_version()}"',
           "-I" + sysconfig.get_paths()["include"], "-I" + os.path.join(torch_dir, "include"),
           "-I" + os.path.join(torch_dir, "include", "torch", "csrc", "api", "include"), "-I/opt/rocm/include", "-o", NATIVE_PATH,
           os.path.join(CSRC, "rtn_native.cpp"), "-L" + os.path.join(torch_dir, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True, cwd=CSRC)
    return NATIVE_PATH


def _native_if_possible(verbose: bool) -> None:
    """The library and its binding work without the native calls, so a missing compiler or header is a warning; an older module does not stay."""
    import warnings
    try:
        if os.path.exists(NATIVE_PATH):
            os.remove(NATIVE_PATH)
        build_native(verbose)
    except (OSError, AttributeError, subprocess.CalledProcessError) as e:
        warnings.warn(f"the binding's native calls were not built ({e}): small calls take 2 us more of host time", RuntimeWarning)


def build_library(verbose: bool = False, extra_flags=()) -> str:
    """Compiles every translation unit (in parallel, objects under _build/) and links the shared library."""
    from concurrent.futures import ThreadPoolExecutor
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    obj_dir = os.path.join(PKG_DIR, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    compile_flags = [f for f in HIPCC_FLAGS if f != "-shared"]

    def compile_one(src):
        obj = os.path.join(obj_dir, src.replace(".hip", ".o"))
        cmd = [hipcc, *compile_flags, *extra_flags, "-c", "-o", obj, os.path.join(CSRC, src)]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True, cwd=CSRC)
        return obj

    with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1)) as pool:
        native = pool.submit(_native_if_possible, verbose)
        objs = list(pool.map(compile_one, SOURCES))
        native.result()
    for name, parts in JOINED.items():
        whole, parts = os.path.join(obj_dir, name), [os.path.join(obj_dir, p) for p in parts]
        subprocess.run(["ld", "-r", "-o", whole + ".joined", *parts], check=True)
        os.replace(whole + ".joined", whole)
        objs = [o for o in objs if o not in parts] + [whole]
    link = [hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB_PATH, *objs]
    if verbose:
        print(" ".join(link), flush=True)
    subprocess.run(link, check=True, cwd=CSRC)
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
