"""Compile the HIP library libnnv.so for gfx950 with hipcc, and the Python module _nnvpy that calls it
with the host compiler (both in-tree, next to this file).  The module needs the interpreter's headers and a
C++ compiler; without it the binding makes the same calls through ctypes."""
from __future__ import annotations

import os
import subprocess
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libnnv.so")
# the suffix names the interpreter and its ABI: another Python does not load what this one built
MODULE = os.path.join(HERE, "_nnvpy" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
SOURCES = ("api.cpp", "cache.cpp", "transform.hip", "direct.hip", "gemm.hip", "winograd.hip")
# packed-fp32 VALU instructions are switched off for every device translation unit
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", INCLUDE, "-I", CSRC]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def build(verbose: bool = False) -> str:
    """Compile every source (always, even if the library exists), link libnnv.so and the module beside it.
    Where the module cannot be built, the library is still complete: a warning, and no module is left over."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    hipcc = _hipcc()

    def compile_one(src: str) -> str:
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc, *FLAGS, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0 or verbose:
            print(" ".join(cmd))
            print(res.stdout, res.stderr)
        if res.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}")
        return obj

    with ThreadPoolExecutor(max_workers=len(SOURCES)) as pool:
        objs = list(pool.map(compile_one, SOURCES))
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        print(res.stdout, res.stderr)
        raise RuntimeError("link failed")
    try:
        build_module(verbose)
    except (RuntimeError, OSError) as e:
        if os.path.exists(MODULE):
            os.remove(MODULE)
        warnings.warn(f"{e}; the binding will call libnnv.so through ctypes")
    return LIB


def build_module(verbose: bool = False) -> str:
    """Compile csrc/pymodule.cpp against the libnnv.so that is there."""
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-I", INCLUDE, "-I", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "pymodule.cpp"), "-o", MODULE, "-L", HERE, "-lnnv", "-Wl,-rpath,$ORIGIN"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0 or verbose:
        print(" ".join(cmd))
        print(res.stdout, res.stderr)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed on pymodule.cpp")
    return MODULE


if __name__ == "__main__":
    print(build(verbose=True))
