"""Builds libtng.so for gfx950 with hipcc and the binding's call extension tng_call.so with g++, in-tree (next to this file).

Flags that matter for reproducible codes: -ffp-contract=off keeps every fp32 operation of the
normalise / threshold / decode path a separately rounded IEEE operation (hipcc would otherwise
contract a*b+c into a fused multiply-add); no fast-math; correctly rounded division (the HIP
default); packed-fp32 instruction selection is switched off.

The sources are compiled side by side (one hipcc process each) into a scratch directory and linked.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtng.so")
CALL = os.path.join(HERE, "tng_call.so")
SOURCES = ["tng_api.hip", "tng_codec.hip", "tng_grad.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-attributes",
]


def call_target() -> str:
    """What the call extension is compiled for, and only used with: its calls depend on the layout of both."""
    import torch

    return f"torch {torch.__version__}, {sys.implementation.cache_tag}"


def call_command() -> list:
    """The compiler line of the call extension: host code against the installed torch and Python headers."""
    import torch

    torch_dir = os.path.dirname(torch.__file__)
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DTNG_BUILT_FOR="{call_target()}"',
            "-isystem", os.path.join(torch_dir, "include"), "-isystem", sysconfig.get_paths()["include"],
            os.path.join(CSRC, "tng_call.cpp"), "-L", os.path.join(torch_dir, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10",
            "-o", CALL]


def build_call(verbose: bool = True) -> bool:
    """Builds the call extension.  Without a compiler or headers for it there is none, and the binding's calls all go through
    ctypes: the same results, 0.5 to 0.7 us of host time more per tensor."""
    try:
        cmd = call_command()
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return True
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        print(f"tng_call.so was not built, calls go through ctypes: {e}", file=sys.stderr, flush=True)
        if os.path.exists(CALL):
            os.remove(CALL)
        return False


def build(verbose: bool = True) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = tempfile.mkdtemp(prefix="libtng_build_")
    try:
        def compile_one(src):
            obj = os.path.join(tmp, src.replace(".hip", ".o"))
            cmd = [hipcc, *FLAGS, "-c", "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj

        with ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as pool:
            call = pool.submit(build_call, verbose)
            objs = list(pool.map(compile_one, SOURCES))
            call.result()
        cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
    finally:
        shutil.rmtree(tmp, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
