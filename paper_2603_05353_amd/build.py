"""Builds libifkv.so (the C-ABI library) in-tree with hipcc for gfx950, and the binding's native
marshalling (host code only).

Usage: python -m paper_2603_05353_amd.build
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "libifkv.so")
MARSHAL_PATH = os.path.join(HERE, "_ifkv_marshal.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 ALU forms are kept out of the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the first kernel arguments arrive in scalar registers with the wavefront instead of by a load at its start, which is the
    # first of the few dependent latencies that a short kernel consists of: 0.1 to 0.4 us a launch (selection of 32K scores
    # 11.9 -> 11.45 us, rotary embedding and splice of 900 rows 10.0 -> 9.3, an fp32 layer of 1024 keys 36.7 -> 36.2; 8 the same)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, src[:-4] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(ln for ln in r.stderr.splitlines() if "packed-fp32-ops" not in ln)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def marshal_command(src: str, out: str) -> list:
    import torch
    from torch.utils import cpp_extension
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    include = [os.path.join(ROOT, "include"), sysconfig.get_paths()["include"], *cpp_extension.include_paths()]
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            *(f"-I{p}" for p in include), src, "-o", out, f"-L{torch_lib}", "-ltorch_python", "-ltorch_cpu", "-lc10"]


def _build_marshal() -> None:
    if os.path.exists(MARSHAL_PATH):
        os.remove(MARSHAL_PATH)   # never one that belongs to other sources
    r = subprocess.run(marshal_command(os.path.join(CSRC, "marshal.cpp"), MARSHAL_PATH), capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("building the marshalling module failed:\n" + r.stderr)


def build_library(jobs: int = 8) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        marshal = ex.submit(_build_marshal)
        objs = list(ex.map(_compile, sources()))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    marshal.result()   # after the library, which serves without it
    return LIB_PATH


if __name__ == "__main__":
    print(build_library())
