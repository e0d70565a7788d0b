"""Builds libspecverify.so (HIP, gfx950 only) with hipcc and the binding's _marshal.so with g++, in-tree.

_marshal.so is host code against the headers of the torch that is installed: it has to be built again for another one.  libspecverify.so has no torch types.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libspecverify.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
# (the slowest to compile first)
SOURCES = ["lm_head_rowmajor.hip", "lm_head_rowmajor_stream.hip", "lm_head_mfma_summary.hip", "lm_head_tile.hip", "lm_head_mfma_buffer.hip", "lm_head_mfma_global.hip", "lm_head_mfma_stream.hip",
           "verify_attn.hip", "lm_head_mfma.hip", "lm_head_packed.hip", "lm_head.hip", "api.hip", "accept.hip", "kv_commit.hip", "assemble_next.hip", "draft_side.hip", "probes.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def build(verbose: bool = False, jobs: int = 7) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        done = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        text = "\n".join(l for l in done.stdout.splitlines() if "packed-fp32-ops" not in l)
        if text.strip():
            sys.stderr.write(text + "\n")
        if done.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}")
        return obj

    with ThreadPoolExecutor(jobs) as pool:                # (a process each; the next starts when one ends)
        objs = list(pool.map(compile_one, SOURCES))
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    build_marshal()
    return LIB


def build_marshal() -> str:
    """The extension module behind binding.py's per-tensor checks (host code, against the headers of the torch that is installed)."""
    import shutil
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths
    if shutil.which("g++") is None:
        raise RuntimeError("the binding's _marshal.so needs g++")
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    include = [x for d in include_paths("cuda") + [sysconfig.get_paths()["include"]] for x in ("-I", d)]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *include, os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL,
           "-L", lib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    subprocess.run(cmd, check=True)
    return MARSHAL


if __name__ == "__main__":
    print(build(verbose=True))
