"""Builds libflexsp.so (HIP, gfx950 only) in-tree with hipcc.

    python -m paper_2412_01523_amd.build [--force]

Each source is compiled to an object under csrc/_build/ (only when it or a header is
newer), then linked into paper_2412_01523_amd/libflexsp.so.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

PKG = Path(__file__).resolve().parent
CSRC = PKG / "csrc"
INCLUDE = PKG.parent / "include"
OBJ = CSRC / "_build"
LIB = PKG / "libflexsp.so"

SOURCES = ["flexsp_host.hip", "pack.hip", "attn_fwd.hip", "attn_fwd_search.hip", "attn_bwd.hip", "attn_bwd_chain.hip", "planner.hip", "fwd_static.hip",
           "lse_merge.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # no NaN is ever produced on a valid path (masked scores are -inf, never inf - inf), so max
    # needs no quieting pass over its inputs: halves the vector work of the row maximum
    "-fno-honor-nans", "-mno-amdgpu-ieee",
    "-Wall", "-Wno-unused-function", f"-I{INCLUDE}", f"-I{CSRC}",
]


# The attention kernels lay out their instruction order by hand (LDS reads issued several matrix
# instructions ahead of their use, softmax arithmetic placed between matrix instructions).  Both
# of the compiler's pre-allocation schedulers otherwise sink every LDS read to just before its
# use, which exposes the full LDS latency once per matrix instruction; with them off the order
# of the source is the order of the code.
SOURCE_ORDER = ["-mllvm", "-pre-RA-sched=source", "-mllvm", "-enable-misched=false"]
# A kernel whose LDS leaves room for one workgroup per compute unit may use all 512 registers, and the compiler then keeps the results of
# matrix instructions in the half that the vector unit cannot read: every score is copied before its exponential.  The
# forward's such kernels need 219 and 253 registers without that half (one had 187 and 96 of it); forwards in halves
# take 5 % less time, whole items in the same kernel 10 % less.  (Kernels that share a compute unit, among them all of the
# backward, are compiled the same either way.)
VECTOR_RESULTS = ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]
PER_SOURCE = {"attn_fwd.hip": SOURCE_ORDER + VECTOR_RESULTS, "attn_fwd_search.hip": SOURCE_ORDER + VECTOR_RESULTS, "attn_bwd.hip": SOURCE_ORDER, "attn_bwd_chain.hip": SOURCE_ORDER}


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    raise RuntimeError("hipcc not found")


def _newest_header() -> float:
    hs = list(CSRC.glob("*.h")) + list(INCLUDE.glob("*.h"))
    return max(h.stat().st_mtime for h in hs)


def _compile(src: str, force: bool, extra) -> Path:
    s = CSRC / src
    o = OBJ / (src + ".o")
    if (not force and o.exists() and o.stat().st_mtime > s.stat().st_mtime
            and o.stat().st_mtime > _newest_header()):
        return o
    cmd = [_hipcc(), *FLAGS, *PER_SOURCE.get(src, []), *extra, "-c", str(s), "-o", str(o)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    # hipcc's host pass does not know the packed-fp32 feature and says so: harmless
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return o


def build_library(force: bool = False, extra_flags=()) -> Path:
    OBJ.mkdir(exist_ok=True)
    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(lambda s: _compile(s, force, list(extra_flags)), SOURCES))
    if force or not LIB.exists() or any(o.stat().st_mtime > LIB.stat().st_mtime for o in objs):
        tmp = LIB.with_suffix(".so.tmp%d" % os.getpid())
        cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc",
               "-o", str(tmp), *map(str, objs)]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed:\n" + r.stderr)
        os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build_library(force="--force" in sys.argv))
