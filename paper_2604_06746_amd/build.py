"""Build libstructkv.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libstructkv.so")
SOURCES = ["api.cpp", "score_mfma_ring.hip", "score_mfma_wide.hip", "score_f32.hip", "score_short.hip", "score_combine.hip", "topk.hip", "gather.hip",
           "aggregate.hip", "pivot.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-x", "hip",
         # packed-fp32 instruction selection is switched off for all device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


# Per-file extras.  The MFMA scoring kernels assume finite inputs (documented in the header): without NaN
# handling the compiler drops the canonicalising v_max it otherwise puts in front of every fmaxf operand.
EXTRA = {"score_mfma_ring.hip": ["-fno-honor-nans"], "score_mfma_wide.hip": ["-fno-honor-nans"]}

# Sources compiled as several objects: (macro that selects the part, number of parts)
PARTS = {"score_mfma_ring.hip": ("SKV_RING_PART", 5)}


def _units() -> list:
    """(source, part) of every object, the sources in parts -- the longest -- first; part is None for a whole source."""
    units = [(s, i) for s in SOURCES if s in PARTS for i in range(PARTS[s][1])]
    return units + [(s, None) for s in SOURCES if s not in PARTS]


def _compile(unit) -> str:
    src, part = unit
    stem = os.path.splitext(src)[0]
    obj = os.path.join(OBJ, stem + (".o" if part is None else "_%d.o" % part))
    define = [] if part is None else ["-D%s=%d" % (PARTS[src][0], part)]
    cmd = ["hipcc"] + FLAGS + EXTRA.get(src, []) + define + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(_compile, _units()))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.run(cmd, check=True)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
