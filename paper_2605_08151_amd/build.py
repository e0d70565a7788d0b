"""Builds libspecverify.so (HIP, gfx950 only) with hipcc and the binding's _marshal.so with g++, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libspecverify.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
# (the slowest to compile first)
SOURCES = ["lm_head_mfma_summary.hip", "lm_head_mfma_buffer.hip", "lm_head_mfma_global.hip", "verify_attn.hip", "lm_head_mfma_stream.hip", "lm_head_rowmajor.hip", "lm_head_tile.hip", "lm_head_mfma.hip", "lm_head_packed.hip", "lm_head.hip", "api.hip", "accept.hip", "kv_commit.hip", "assemble_next.hip", "draft_side.hip", "probes.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def build(verbose: bool = False, jobs: int = 5) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        if len(procs) >= jobs:
            _drain(procs)
    _drain(procs)
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    build_marshal()
    return LIB


def build_marshal() -> str:
    """The extension module behind binding.py's per-tensor checks (host code, against the headers of the torch that is installed)."""
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    include = [x for d in include_paths("cuda") + [sysconfig.get_paths()["include"]] for x in ("-I", d)]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *include, os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL,
           "-L", lib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    subprocess.run(cmd, check=True)
    return MARSHAL


def _drain(procs):
    while procs:
        src, p = procs.pop(0)
        out, _ = p.communicate()
        text = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            sys.stderr.write(text + "\n")
            raise RuntimeError(f"hipcc failed on {src}")
        if text.strip():
            sys.stderr.write(text + "\n")


if __name__ == "__main__":
    print(build(verbose=True))
