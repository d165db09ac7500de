"""Compile libfastgl_agg.so for gfx950 with hipcc, and _host.so (the native marshalling of its calls for
Python) with g++; both in-tree, next to this file."""
from __future__ import annotations

import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libfastgl_agg.so")
HOST = os.path.join(HERE, "_host.so")
SOURCES = ["api.hip", "bookkeeping.hip", "aggregate.hip", "update.hip", "update_narrow.hip", "update_rows.hip", "idmap.hip", "match.hip", "overlap.hip", "edge.hip",
           "static_scratch.hip", "layer.hip"]


def build_library(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
           # packed-fp32 instruction selection is switched off for all device code
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(HERE, "csrc")]
    cmd += [os.path.join(HERE, "csrc", s) for s in SOURCES]
    cmd += ["-o", LIB]
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err)
    return LIB


def build_host(verbose: bool = False) -> str:
    """Links against libfastgl_agg.so, so that is built first."""
    import torch
    site = os.path.dirname(os.path.abspath(torch.__file__))
    inc = [os.path.join(ROOT, "include"), sysconfig.get_paths()["include"], os.path.join(site, "include"),
           os.path.join(site, "include", "torch", "csrc", "api", "include"), "/opt/rocm/include"]
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *["-I" + d for d in inc],
           os.path.join(HERE, "csrc", "host.cpp"), "-o", HOST, "-L" + HERE, "-lfastgl_agg",
           "-L" + os.path.join(site, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + res.stderr)
    if verbose and res.stderr.strip():
        print(res.stderr)
    return HOST


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_host(verbose=True))
