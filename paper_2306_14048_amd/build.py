"""Builds libh2o_hip.so (the C-ABI library) in-tree with hipcc for gfx950, and the
native part of the Python binding (_step_call.so, host code) with g++.

    python -m paper_2306_14048_amd.build

hipcc cross-compiles without a GPU.  The packed-fp32 instructions are disabled
for the device pass on purpose (build flag below); the host pass warns that it
does not know that feature, which is harmless.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libh2o_hip.so")
STEP_CALL = os.path.join(PKG, "_step_call.so")
OBJ_DIR = os.path.join(PKG, "_build")
SOURCES = ["h2o_api.hip", "decode_step.hip", "decode_step_q4.hip", "decode_split.hip", "prefill_scores.hip", "prefill_attention.hip",
           "select_gather.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    "-Wall", "-Wno-unused-command-line-argument",
]


def _compile(src: str, extra) -> str:
    obj = os.path.join(OBJ_DIR, src.replace(".hip", ".o"))
    cmd = ["hipcc", *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _build_step_call() -> None:
    import torch
    from torch.utils import cpp_extension
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    rocm = cpp_extension.ROCM_HOME or "/opt/rocm"
    inc = [os.path.join(ROOT, "include"), sysconfig.get_paths()["include"], os.path.join(rocm, "include"),
           *cpp_extension.include_paths()]
    tmp = STEP_CALL + ".tmp%d" % os.getpid()
    subprocess.check_call(
        ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-Wall", "-D__HIP_PLATFORM_AMD__",
         "-DUSE_ROCM", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI]
        + [x for i in inc for x in ("-isystem", i)]
        # (-z now: another torch without one of its symbols fails the import, not a step)
        + [os.path.join(CSRC, "step_call.cpp"), "-o", tmp, "-L", PKG, "-l:libh2o_hip.so", "-Wl,-rpath,$ORIGIN", "-Wl,-z,now", "-L", lib,
           "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"])
    os.replace(tmp, STEP_CALL)


def build(extra_flags=(), verbose: bool = True) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), SOURCES))
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    _build_step_call()
    if verbose:
        print("built", LIB, STEP_CALL)
    return LIB


if __name__ == "__main__":
    build(sys.argv[1:])
