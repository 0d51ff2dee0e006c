"""Builds libmtla.so for gfx950 with hipcc (in-tree, next to this file)."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmtla.so")
SOURCES = ["mtla_api.hip", "append.hip", "attn_valu.hip", "attn_f32.hip", "attn_mfma.hip", "attn_cols.hip", "attn_whole.hip", "proj.hip", "combine_mfma.hip", "prefill_front.hip", "prefill_explicit.hip", "gemm_wide.hip", "gemm_ring.hip", "prefill_latent.hip", "layer.hip", "pages.hip"]
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-fno-gpu-rdc", "-Wall", "-Wno-unused-function",
    # no packed fp32 instructions: hipcc makes them out of ordinary float code, and some of their forms have given wrong results
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


PYCALL = os.path.join(HERE, "_mtla_call.so")  # native call path of the Python binding (host code, CPython API)


def pycall_command() -> list:
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    return (["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Wno-unused-function",
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", os.path.join(CSRC, "pycall.cpp")]
            + [f"-isystem{d}" for d in cpp_extension.include_paths()] + [f"-I{sysconfig.get_paths()['include']}", "-o", PYCALL]
            + [f"-L{d}" for d in cpp_extension.library_paths()] + ["-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10"])


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found: libmtla needs the ROCm toolchain")
    return exe


def build_library(verbose: bool = True) -> str:
    """Compile every HIP source into paper_2505_13544_amd/libmtla.so, and the binding's native call path beside it."""
    objs = []
    obj_dir = os.path.join(HERE, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    procs = []
    for src in SOURCES:
        obj = os.path.join(obj_dir, src.replace(".hip", ".o"))
        cmd = [hipcc()] + [f for f in HIPCC_FLAGS if f != "-shared"] + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print("[build]", " ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    cmd = pycall_command()
    if verbose:
        print("[build]", " ".join(cmd), flush=True)
    procs.append(("pycall.cpp", subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if out.strip() and verbose:
            print(out)
        if p.returncode != 0:
            raise RuntimeError(f"the compiler failed on {src}:\n{out}")
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    if verbose:
        print("[build]", " ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build_library())
    sys.exit(0)
