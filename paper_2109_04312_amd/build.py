"""Builds csrc/*.hip into libmate.so (gfx950) and csrc/bind.cpp into _native.so (host code over torch's
headers) next to this file.  `python -m paper_2109_04312_amd.build`."""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmate.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["api.hip", "segments.hip", "positions.hip", "probe.hip", "proj_mfma.hip", "attn_f32_mfma.hip", "attn_fwd_mfma.hip", "attn_bwd_mfma.hip", "attn_dense_mfma.hip"]
# packed-fp32 instructions are switched off on purpose (device code only).  Kernel arguments that are plain values arrive in
# registers with the wavefront instead of by its first load (builder and cell positions: 0.2 us a launch).
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature",
         "-Xclang", "-packed-fp32-ops", "-mllvm", "-amdgpu-mfma-vgpr-form", "-mllvm", "-amdgpu-kernarg-preload-count=14", "-fno-honor-nans", "-Wall", "-Wno-unused-function", "-Wno-inline-asm"]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        print(err, file=sys.stderr)
    return obj


def _bind() -> None:
    import torch
    from torch.utils import cpp_extension
    inc = [f"-I{p}" for p in (*cpp_extension.include_paths(), "/opt/rocm/include", sysconfig.get_paths()["include"])]
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *inc, os.path.join(CSRC, "bind.cpp"),
           "-o", NATIVE, f"-L{lib}", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch", "-ltorch_python"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for bind.cpp:\n" + r.stderr)


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        native = ex.submit(_bind)
        objs = list(ex.map(_compile, SOURCES))
        native.result()
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print("built", LIB, NATIVE)
    return LIB


if __name__ == "__main__":
    build()
