"""Builds libgsd.so (the gfx950 HIP library behind include/gsd.h) in-tree with hipcc, and the native part of its Python binding."""
from __future__ import annotations

import hashlib
import importlib.machinery
import os
import subprocess
import sysconfig

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libgsd.so")
BINDING_PATH = os.path.join(PKG_DIR, "_binding" + importlib.machinery.EXTENSION_SUFFIXES[0])
BENCH_LIB_PATH = os.path.join(PKG_DIR, "libgsd_bench.so")     # measurement aid of bench.py only

SOURCES = ["gsd_api.hip", "mask_build.hip", "accept_path.hip", "node_argmax.hip", "dag_attention_f32.hip",
           "dag_attention_bf16.hip", "dag_attention_bf16_keys.hip", "unmerge_tree.hip", "commit_kv.hip", "accept_stochastic.hip", "build_graph.hip"]

# -no-hip-rt: the library carries no dependency on a particular libamdhip64; the process that loads it (the
# Python binding: the runtime torch already runs on) supplies the HIP runtime.  Two HIP runtimes in one process
# do not share devices, streams or pointers.
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-no-hip-rt",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall",
               "-Wno-unused-command-line-argument"]


def header_id() -> str:
    """Identity of gsd.h, compiled into the library and into the binding's native part: whether they go together."""
    with open(os.path.join(ROOT, "include", "gsd.h"), "rb") as f:
        return hashlib.sha256(f.read()).hexdigest()[:16]


def build_binding(verbose: bool = False) -> str | None:
    """csrc/binding.cpp against the headers of the torch that is installed; host code only.  The library does not need it, nor
    does the Python binding: where it cannot be built (no torch, no compiler, no headers) a line says so, none is left behind
    from an earlier build, and None is returned."""
    if os.path.exists(BINDING_PATH):
        os.remove(BINDING_PATH)
    try:
        cmd = _binding_command()
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        print(f"{os.path.basename(BINDING_PATH)} was not built ({e}): Python calls go without it, which takes them longer", flush=True)
        return None
    return BINDING_PATH


def _binding_command() -> list[str]:
    import torch
    from . import built_for
    root = os.path.dirname(torch.__file__)
    headers = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
               sysconfig.get_paths()["include"]]
    lib = os.path.join(root, "lib")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-Wno-sign-compare",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DGSD_BUILT_FOR="{built_for(torch, header_id())}"',
            *[flag for path in headers for flag in ("-isystem", path)], "-I", os.path.join(ROOT, "include"),
            os.path.join(CSRC, "binding.cpp"), "-o", BINDING_PATH, "-L", lib, "-lc10", "-ltorch_cpu", "-ltorch_python",
            f"-Wl,-rpath,{lib}"]


def build_library(verbose: bool = False, extra_flags: list[str] | None = None) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *(extra_flags or []), f'-DGSD_HEADER_ID="{header_id()}"', "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB_PATH]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    cmd = [hipcc, *HIPCC_FLAGS, *(extra_flags or []), os.path.join(CSRC, "bench_mfma_loop.hip"), "-o", BENCH_LIB_PATH]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    build_binding(verbose)
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
