"""Builds libmxq.so (hand-written HIP kernels for gfx950 + the C ABI) in-tree with hipcc, and _mxq_calls.so (the
native calls of the Python binding, host code on torch's C++ interface) with g++."""
from __future__ import annotations

import hashlib
import os
import subprocess
import sys
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libmxq.so")
CALLS = os.path.join(_HERE, "_mxq_calls.so")
SOURCES = ["mxq_api.hip", "stream_kernels.hip", "brute_kernels.hip", "aux_kernels.hip", "diag_kernels.hip"]

# No fast-math and no FMA contraction: every rounding in the kernels is written out.
# Packed-fp32 instructions are switched off for the device compiler.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
         "-ffp-contract=off", "-fno-fast-math",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument"]


def _run(cmd, verbose):
    try:
        res = subprocess.run(cmd, capture_output=True, text=True)
    except FileNotFoundError:
        raise RuntimeError(f"{cmd[0]} is not installed") from None
    if verbose or res.returncode != 0:
        print(res.stdout)
        print(res.stderr)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed: " + " ".join(cmd))


def header_id() -> str:
    """Identity of include/mxq.h, compiled into both libraries: the native calls take libmxq's functions by address."""
    with open(os.path.join(os.path.dirname(_HERE), "include", "mxq.h"), "rb") as f:
        return hashlib.sha256(f.read()).hexdigest()[:16]


def calls_abi() -> str:
    """The interpreter and the torch, to the commit, whose layouts are compiled into _mxq_calls.so (mxq.py compares it)."""
    import torch
    return f"{sys.implementation.cache_tag} {torch.__version__} {torch.version.git_version}"


def _calls_command():
    import torch
    root = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            f'-DMXQ_CALLS_ABI="{calls_abi()}"', f'-DMXQ_HEADER_ID="{header_id()}"',
            "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include/torch/csrc/api/include"),
            "-isystem", os.path.join(rocm, "include"), "-isystem", sysconfig.get_paths()["include"],
            os.path.join(CSRC, "binding.cpp"), "-o", CALLS, "-L" + os.path.join(root, "lib"),
            "-ltorch_python", "-ltorch_hip", "-ltorch_cpu", "-lc10_hip", "-lc10"]


def build_calls(verbose: bool = False) -> str | None:
    """Builds _mxq_calls.so; None without torch, whose interface it is for (and without which nothing loads it)."""
    try:
        cmd = _calls_command()
    except ImportError:
        return None
    _run(cmd, verbose)
    return CALLS


def build_library(verbose: bool = False, jobs: int = 4) -> str:
    """Compiles every translation unit (in parallel), links libmxq.so and builds _mxq_calls.so next to this file.
    The C library needs hipcc only: it is linked before anything that the native calls lack is reported."""
    with tempfile.TemporaryDirectory(prefix="mxq_build_") as tmp, ThreadPoolExecutor(max_workers=max(1, jobs)) as pool:
        objs = [os.path.join(tmp, s.replace(".hip", ".o")) for s in SOURCES]
        cmds = [["hipcc", *FLAGS, f'-DMXQ_HEADER_ID="{header_id()}"', "-c", os.path.join(CSRC, s), "-o", o]
                for s, o in zip(SOURCES, objs)]
        units = [pool.submit(_run, c, verbose) for c in cmds]
        calls = pool.submit(build_calls, verbose)
        for u in units:
            u.result()
        _run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-fvisibility=hidden", *objs, "-o", LIB],
             verbose)
        calls.result()
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
