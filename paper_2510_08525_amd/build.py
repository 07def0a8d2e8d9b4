"""Builds librlkv.so (HIP kernels + C-ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "librlkv.so")
OBJ_DIR = os.path.join(PKG, "_build")

SOURCES = ["rlkv_api.hip", "append_evict.hip", "worklist_combine.hip", "decode_valu.hip", "decode_mfma.hip",
           "prefill_mfma.hip", "stream_probe.hip", "share_plan.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-Wall",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    # without the packed-fp32 VALU forms: every test and figure of the library is of code compiled like this
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


# Per-file additions: the prefill kernel's maxima need no NaN quieting (see the comment there), and its hot loop wants to begin on
# a cache line: the same instructions a few bytes further on took 0.8 % longer (16 x 16 384 tokens, 15.68 against 15.57 ms).
# The first 14 words of a kernel's arguments in scalar registers before its first instruction: of kernels whose start is a chain of
# memory latencies (see decode_mfma.hip).
PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=14"]
EXTRA_FLAGS = {"decode_mfma.hip": PRELOAD, "decode_valu.hip": PRELOAD, "worklist_combine.hip": PRELOAD,
               "prefill_mfma.hip": ["-fno-honor-nans", "-falign-loops=64"]}


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *HIPCC_FLAGS, *EXTRA_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "not a recognized feature" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build_library(verbose: bool = True) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stderr)
    if verbose:
        print(f"built {LIB}")
    return LIB


EXAMPLE_SRC = os.path.join(ROOT, "examples", "c_abi_decode.c")
EXAMPLE_BIN = os.path.join(ROOT, "examples", "c_abi_decode")


def build_example(verbose: bool = True) -> str:
    """The plain-C program under examples/ that drives the library through include/rlkv.h alone (host compiler,
    C11): built against the library just linked, found at run time relative to the binary."""
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = [os.environ.get("CC", "gcc"), "-std=c11", "-O2", "-Wall", "-D__HIP_PLATFORM_AMD__",
           "-I", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"), EXAMPLE_SRC,
           "-L", PKG, "-lrlkv", "-L", os.path.join(rocm, "lib"), "-lamdhip64", "-lm",
           "-Wl,-rpath,$ORIGIN/../paper_2510_08525_amd", "-Wl,-rpath," + os.path.join(rocm, "lib"), "-o", EXAMPLE_BIN]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("building the C example failed:\n" + res.stderr)
    if verbose:
        print(f"built {EXAMPLE_BIN}")
    return EXAMPLE_BIN


if __name__ == "__main__":
    build_library()
    build_example()
