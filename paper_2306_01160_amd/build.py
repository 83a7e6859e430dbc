"""Builds libscfa.so (HIP, gfx950 only) next to this file.

    python -m paper_2306_01160_amd.build

hipcc cross-compiles without a GPU.  Every translation unit is compiled on its own
(in parallel) and the objects are linked into one shared library.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libscfa.so")

SOURCES = ["scfa_api.hip", "scfa_index.hip", "scfa_lsh.hip", "scfa_ranges.hip", "scfa_attn_f32.hip", "scfa_attn_fwd.hip",
           "scfa_attn_bwd.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 VALU forms are kept off on this machine pool
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # keep MFMA accumulators in VGPRs (no accumulation-register copies around the softmax)
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
    # no kernel forms a NaN whose value it uses (masked scores are -inf, never inf - inf; the pieces of an infinite
    # fp32 number are, and its item is left to kernel code without pieces); this lets max/min skip the quieting of
    # signalling NaNs.  Where an input may be one, its bits are tested, behind an empty asm that hides them.
    "-fno-honor-nans",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# the argument checks of the C ABI test for NaN: that file keeps IEEE semantics
HONOR_NANS = {"scfa_api.hip"}


def _compile(src: str, extra) -> str:
    obj = os.path.join(OBJ_DIR, src.replace(".hip", ".o"))
    flags = [f for f in FLAGS if not (src in HONOR_NANS and f == "-fno-honor-nans")]
    cmd = [HIPCC, *flags, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass warns that it does not know the packed-fp32 feature: harmless
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = False, extra_flags=(), lib: str = LIB) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stderr)
    if verbose:
        print(lib)
    return lib


if __name__ == "__main__":
    extra = [a for a in sys.argv[1:] if a.startswith("-")]
    out = [a for a in sys.argv[1:] if not a.startswith("-")]
    build(verbose=True, extra_flags=extra, lib=out[0] if out else LIB)
