"""Build libpcls.so (gfx950) in-tree with hipcc.

    python -m paper_2606_06656_amd.build

Every HIP source is compiled with packed-FP32 instructions disabled (the
compiler would otherwise form v_pk_* FP32 operations from scalar code).
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpcls.so")
SOURCES = ["pcls.hip", "plan.cpp", "mpnn.hip", "mpnn_net.hip"]
ARCH = os.environ.get("PCLS_OFFLOAD_ARCH", "gfx950")

HIP_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # work claims are single-lane atomics on one LDS word: the pass that turns
    # uniform-address atomics into a wave reduction only adds instructions there
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
    "-Wall", "-Wno-unused-function",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    return "hipcc"


def objects():
    """(object name, source, extra flags) of every compilation: the variants of the
    engine's kernels are compiled side by side."""
    out = []
    for maxb in ("kMaxbAll", "kMaxbMid", "kMaxbShort"):
        for bits, acc in ((32, "unsigned int"), (64, "unsigned long long")):
            # PCLS_VARIANT_LT: log2 of the restarts per tile, -1 any; -2 the batched
            # engine, -3 the statistics, -4 codes in LDS, -5 the same problems without
            # (-6 in the batched engine)
            kinds = [-1, 0, -2] + ([-3] if bits == 32 else []) + ([1, 2, -4, -5, -6] if maxb == "kMaxbShort" else [])
            for lt in kinds:
                out.append((f"pcls_{maxb}_{bits}_{lt}.o", "pcls.hip",
                            [f"-DPCLS_VARIANT_MAXB={maxb}", f"-DPCLS_VARIANT_ACC={acc}", f"-DPCLS_VARIANT_LT={lt}"]))
    return out + [(src.rsplit(".", 1)[0] + ".o", src, []) for src in SOURCES]


def build(verbose: bool = False) -> str:
    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            sys.stderr.write(res.stdout + res.stderr)
            raise RuntimeError("hipcc failed building libpcls.so")

    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as work, ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
        jobs = [(os.path.join(work, o), os.path.join(CSRC, src), flags) for o, src, flags in objects()]
        list(pool.map(lambda j: run([hipcc(), *HIP_FLAGS, *j[2], "-c", j[1], "-o", j[0]]), jobs))
        run([hipcc(), f"--offload-arch={ARCH}", "-fPIC", "-shared", "-o", tmp, *(j[0] for j in jobs)])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
