"""Compile the HIP sources into the in-tree shared library (gfx950 only)."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libquasar.so")
FAST = os.path.join(HERE, "_fastcall.so")
SOURCES = ["quasar_api.hip", "direct_int8.hip", "direct_bf16.hip", "direct_w8a8.hip", "direct_w4.hip",
           "outer_w8a8.hip", "outer_w4.hip"]
HEADERS = ["quasar_device.hpp", "launch.hpp", "shares.hpp", "stream_gemm.hpp", "stream_direct.hpp", "stream_direct_a8.hpp", "stream_direct_w4.hpp", "stream_outer.hpp", "norm.hpp", "stream_sequence.hpp", "stream_w8a8.hpp", "stream_w4.hpp", "drafter.hpp", "attention.hpp", "sample.hpp", "draw.hpp", "pack.hpp", "probe.hpp", "unlocked.hpp"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 vector instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the whole-step kernel keeps rarely executed phase-entry code inside a fully unrolled round;
    # without this the compiler silently refuses "#pragma unroll" once that body grows
    "-mllvm", "-pragma-unroll-threshold=1000000",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def build_library(verbose: bool = False, extra_flags=()) -> str:
    """Compiles the sources side by side and links them."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    # the binding's argument marshalling (host code, against torch's headers)
    fast = [os.environ.get("CXX") or "g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            *("-I" + d for d in cpp_extension.include_paths()), "-I" + sysconfig.get_paths()["include"], "-o", FAST, os.path.join(CSRC, "fastcall.cpp"),
            *("-L" + d for d in cpp_extension.library_paths()), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, src + ".o") for src in SOURCES]
        jobs = [[hipcc(), *HIPCC_FLAGS, *extra_flags, "-c", "-o", obj, os.path.join(CSRC, src)]
                for src, obj in zip(SOURCES, objects)] + [fast]
        link = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objects]
        with ThreadPoolExecutor(max_workers=len(jobs)) as pool:
            for _ in pool.map(lambda cmd: _run(cmd, verbose), jobs):
                pass
        _run(link, verbose)
    return LIB


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed:\n{res.stdout}")
    lines = [l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l and l.strip()]
    if verbose and lines:
        print("\n".join(lines), flush=True)


if __name__ == "__main__":
    print(build_library(verbose=True, extra_flags=sys.argv[1:]))
