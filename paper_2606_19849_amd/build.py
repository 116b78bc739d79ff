"""Compile libvico.so (HIP kernels + C ABI) and the measurement helper
libvico_bench.so for gfx950, and the binding's C++ calls (_vico_call.so),
in-tree.

Usage: python -m paper_2606_19849_amd.build   (or build() from Python)
"""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libvico.so")
SOURCES = ["attn_fwd.hip", "attn_merge.hip", "attn_gather.hip", "attn_rows.hip", "retrieve.hip", "token_drop.hip", "kv_append.hip", "vico_api.hip", "noalloc.hip"]
BENCH_LIB = os.path.join(PKG, "libvico_bench.so")
BENCH_SOURCES = ["mfma_peak.hip"]

CALL_LIB = os.path.join(PKG, "_vico_call.so")
CALL_SOURCE = "py_call.cpp"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-mcode-object-version=5",
    # keep hipcc from emitting packed fp32 VALU ops (v_pk_*_f32)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-unused-result",
]


def build(verbose: bool = False, extra_flags=()) -> str:
    """Compile libvico.so, libvico_bench.so and _vico_call.so; return the path of libvico.so."""
    _compile(SOURCES, LIB, verbose, extra_flags)
    _compile(BENCH_SOURCES, BENCH_LIB, verbose, extra_flags)
    _compile_calls(verbose)
    return LIB


def _compile_calls(verbose) -> None:
    """The binding's C++ calls: host code against torch's headers and libvico.so."""
    import sysconfig

    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    tmp = CALL_LIB + ".tmp"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", INCLUDE, "-I", inc,
           "-I", os.path.join(inc, "torch", "csrc", "api", "include"), "-I", sysconfig.get_paths()["include"],
           "-I", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), os.path.join(CSRC, CALL_SOURCE),
           "-o", tmp, "-L", PKG, "-l:libvico.so", "-L", os.path.join(os.path.dirname(torch.__file__), "lib"),
           "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed ({res.returncode}):\n{res.stderr}")
    os.replace(tmp, CALL_LIB)


def _compile(sources, lib, verbose, extra_flags) -> None:
    srcs = [os.path.join(CSRC, s) for s in sources]
    tmp = lib + ".tmp"
    cmd = [HIPCC, *FLAGS, *extra_flags, "-I", INCLUDE, "-I", CSRC, *srcs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 feature and says so; that is expected
    noise = "'-packed-fp32-ops' is not a recognized feature"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{err}")
    if verbose and err.strip():
        print(err, file=sys.stderr)
    # A kernel whose host-side launch stub was not emitted links into an
    # unloadable library; refuse it here instead of at load time.
    nm = subprocess.run(["nm", "-u", tmp], capture_output=True, text=True)
    missing = [l.split()[-1] for l in nm.stdout.splitlines() if "__device_stub__" in l]
    if missing:
        raise RuntimeError(f"{os.path.basename(lib)} references kernel stubs that were not emitted: {missing}")
    os.replace(tmp, lib)


if __name__ == "__main__":
    print(build(verbose=True))
