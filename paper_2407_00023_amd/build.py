"""Build libprefixattn.so for gfx950 with hipcc, and the Python module of the hot-path calls with g++ (in-tree, next to
this file)."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libprefixattn.so")
CALLS = os.path.join(HERE, "_calls.so")
SOURCES = ["tree.cpp", "sched.cpp", "profile.cpp", "call_sets.cpp", "tree_changes.hip", "match.hip", "kvpool.hip", "extend.cpp", "extend_f32.hip", "extend_plan.hip", "extend_bf16.hip", "calib.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 code generation
         "-Wall", "-Wno-unused-function"]


# extend_bf16.hip never produces or consumes a NaN on purpose (the -inf cases are guarded explicitly), so
# the compiler may drop the NaN-quieting copies it otherwise puts in front of every fmaxf
EXTRA_FLAGS = {"extend_bf16.hip": ["-fno-honor-nans"]}


def _hipcc() -> str:
    for c in ("/opt/rocm/bin/hipcc", "hipcc"):
        if os.path.sep not in c or os.path.exists(c):
            return c
    return "hipcc"


def _compile_calls() -> str:
    """The host-only Python module _calls (csrc/calls.cpp) against the torch that is installed."""
    import torch
    t = os.path.dirname(torch.__file__)
    obj = os.path.join(OBJ, "calls.o")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
                           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                           "-I" + os.path.join(t, "include"), "-I" + os.path.join(t, "include", "torch", "csrc", "api", "include"),
                           "-I/opt/rocm/include", "-I" + sysconfig.get_paths()["include"],
                           "-c", os.path.join(CSRC, "calls.cpp"), "-o", obj])
    return obj


def _link_calls(obj: str) -> None:
    import torch
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    subprocess.check_call(["g++", "-shared", "-fPIC", obj, "-o", CALLS, "-L" + HERE, "-l:libprefixattn.so", "-L" + lib, "-lc10",
                           "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-Wl,-rpath,$ORIGIN"])


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    hipcc = _hipcc()
    # the assembly of the steady-state tile runs is written by a generator that sits beside the sources
    subprocess.check_call([sys.executable, os.path.join(CSRC, "gen_fast_run.py")], stdout=subprocess.DEVNULL)

    def compile_one(src):
        obj = os.path.join(OBJ, src.rsplit(".", 1)[0] + ".o")
        cmd = [hipcc] + FLAGS + EXTRA_FLAGS.get(src, []) + ["-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{err}")
        if verbose and err.strip():
            print(err, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=8) as ex:
        calls = ex.submit(_compile_calls)
        objs = list(ex.map(compile_one, SOURCES))
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    _link_calls(calls.result())
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
