"""Builds libspecdraft.so (HIP, gfx950 only) in-tree with hipcc.

    python -m paper_2404_19124_amd.build

Every translation unit is compiled on its own (in parallel) and linked into
paper_2404_19124_amd/libspecdraft.so.  No JIT, no cache outside the tree.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libspecdraft.so")

CALL = os.path.join(HERE, "_call.so")   # the binding's native half (host code, against torch's headers)

SOURCES = [
    "spec_lib.hip",
    "kernels_stage.hip",
    "kernels_verify.hip",
    "kernels_f32.hip",
    "kernels_head_skinny.hip",
    "kernels_head_skinny32.hip",
    "kernels_head_gemm.hip",
    "kernels_head_tile.hip",
    "kernels_head_panel.hip",
    "kernels_head_once.hip",
    "kernels_tree_meta.hip",
]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


# Per-file additions.  The dense contraction keeps its accumulators in VGPRs: with the
# default heuristic the register allocator shuffles 128 accumulators between AGPRs and
# VGPRs on every loop trip.
EXTRA = {"kernels_head_gemm.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = [hipcc(), *FLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _compile_call() -> None:
    import torch
    root = os.path.dirname(torch.__file__)
    inc = os.path.join(root, "include")
    cmd = [shutil.which("g++") or "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-isystem", inc,
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "call.cpp"), "-o", CALL,
           # (loaded by `import torch` already: no search path of its own)
           "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for call.cpp:\n" + r.stderr)
    if r.stderr.strip():
        sys.stderr.write(r.stderr)


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        call = ex.submit(_compile_call)
        objs = list(ex.map(_compile, SOURCES))
        call.result()
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
