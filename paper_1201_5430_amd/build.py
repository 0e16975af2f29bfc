"""Build liblhfmm.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblhfmm.so")
SOURCES = ["lhf_plan.hip", "lhf_eval.hip", "lhf_m2l.hip", "lhf_m2l_half.hip", "lhf_m2l_quarter.hip",
           "lhf_m2l_turn.hip", "lhf_m2l_mfma.hip", "lhf_batch.hip", "lhf_filament.hip"]
# compiled once per type and order: whole vectors per lane, vectors split over a wavefront's rows
TURN = [("m2l_turn", "double", p) for p in range(7, 13)] + [("m2l_turn", "float", p) for p in range(7, 17)] + \
    [("m2l_rows", "double", p) for p in range(13, 25)] + \
    [("mm_rows", "double", p) for p in range(7, 25)] + [("mm_rows", "float", p) for p in range(7, 17)]
ARCH = os.environ.get("LHF_OFFLOAD_ARCH", "gfx950")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared", f"--offload-arch={ARCH}",
    # no packed-FP32 instructions in any device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


# per-source additions: the half-vector M2L's fully unrolled FP32 p = 16 body exceeds the
# default size limit of '#pragma unroll' (a partly rolled loop would move its vectors to scratch)
EXTRA = {"lhf_m2l_half.hip": ["-mllvm", "-pragma-unroll-threshold=200000"],
         "lhf_m2l_quarter.hip": ["-mllvm", "-pragma-unroll-threshold=200000"]}


def units():
    """(object, source, extra flags) of every compilation, the longest first"""
    out = [(f"lhf_{k}_{t}_{p}.o", f"lhf_{k}_p.hip", [f"-DLHF_TURN_T={t}", f"-DLHF_TURN_P={p}"])
           for k, t, p in sorted(TURN, key=lambda u: -u[2])]
    rest = [(s.replace(".hip", ".o"), s, EXTRA.get(s, [])) for s in SOURCES]
    return sorted(rest, key=lambda u: u[1] not in EXTRA)[:len(EXTRA)] + out + \
        sorted(rest, key=lambda u: u[1] not in EXTRA)[len(EXTRA):]


def _headers(src: str, seen=None) -> set:
    """the quoted includes of a source, followed through"""
    seen = set() if seen is None else seen
    for h in re.findall(r'#include "([^"]+)"', open(src).read()):
        f = os.path.normpath(os.path.join(os.path.dirname(src), h))
        if f not in seen and os.path.exists(f):
            seen.add(f)
            _headers(f, seen)
    return seen


def _stale(obj: str, src: str) -> bool:
    """True if obj is missing or older than its source or a header that it includes."""
    if not os.path.exists(obj):
        return True
    t = os.path.getmtime(obj)
    return any(os.path.getmtime(d) > t for d in [src, *_headers(src)])


def build(verbose: bool = False, jobs: int = 0, incremental: bool = False) -> str:
    """Compile every source (in parallel, at most ``jobs`` at once) and link liblhfmm.so.

    incremental=True recompiles only the objects that are older than their source or a header.
    """
    from concurrent.futures import ThreadPoolExecutor
    objs, cmds = [], []
    for o, src, extra in units():
        obj, src = os.path.join(CSRC, o), os.path.join(CSRC, src)
        objs.append(obj)
        if incremental and not _stale(obj, src):
            continue
        cmds.append(["hipcc", "-c", *[f for f in FLAGS if f != "-shared"], *extra, "-o", obj, src])

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)

    jobs = jobs or max(1, min(len(cmds), 8, os.cpu_count() or 1))
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        for f in [ex.submit(run, c) for c in cmds]:
            f.result()
    tmp = LIB + ".tmp"
    cmd = ["hipcc", "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv, incremental="-i" in sys.argv))
