"""Build libmlm_shard.so (HIP, gfx950 only) in-tree with hipcc.

    python -m paper_1909_08053_amd.build          # compile every translation unit, link
Every source is compiled on each call (object files are rebuilt, in parallel); the shared
library lands next to this file so that it travels with the tree.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmlm_shard.so")
MODULE = os.path.join(HERE, "_mlm_call.so")

SOURCES = ["api.hip", "rowops.hip", "gemm_f32.hip", "gemm_f32_pieces.hip", "attention_f32.hip", "gemm_bf16.hip",
           "gemm_bf16_fwd.hip", "gemm_bf16_dgrad.hip", "gemm_bf16_wgrad.hip", "gemm_bf16_dual.hip", "attention_bf16.hip", "optimizer.hip", "embed.hip"]

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = [_hipcc(), *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _module() -> None:
    """The CPython module that marshals the hot calls' arguments; host code against torch's headers, linked to the library beside it."""
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    root = os.path.dirname(torch.__file__)
    inc = [f"-I{d}" for d in [os.path.join(ROOT, "include"), sysconfig.get_paths()["include"], *cpp_extension.include_paths(),
                               os.path.join(cpp_extension.ROCM_HOME or "/opt/rocm", "include")]]
    cmd = [_hipcc(), "--offload-arch=gfx950", "-x", "c++", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM", "-O2", "-std=c++17", "-fPIC", "-shared",
           "-fvisibility=hidden", "-w", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *inc,
           os.path.join(CSRC, "py_call.cpp"), "-o", MODULE, f"-L{HERE}", "-l:libmlm_shard.so", "-Wl,-rpath,$ORIGIN", f"-L{root}/lib",
           "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("py_call.cpp failed:\n" + r.stderr)


def build(jobs: int = 8, verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    if os.path.exists(MODULE):
        os.remove(MODULE)                # (an older one would marshal by the signatures of an older library)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    try:
        _module()
    except (ImportError, OSError, RuntimeError) as e:
        # the binding does the same through ctypes, some 30 us of host time a step of 40 launches slower
        sys.stderr.write(f"{os.path.basename(MODULE)} is not built, arguments will go through ctypes: {e}\n")
    if verbose:
        print(f"built {LIB} ({os.path.getsize(LIB) / 1e6:.1f} MB)")
    return LIB


if __name__ == "__main__":
    build()
