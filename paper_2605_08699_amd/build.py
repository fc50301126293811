"""Builds libtigas.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtigas.so")
SOURCES = ["kernels.hip", "jpeg.hip", "api.cpp", "registry.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # the FP32 operation sequence is written out explicitly (fmaf where fused)
    "-ffp-contract=off",
    # no packed-FP32 instructions (v_pk_*_f32)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]


# the compiler's report of each kernel's registers, spills and scratch memory
REPORT = ["-Rpass-analysis=kernel-resource-usage"]


def spilling_kernels(report: str):
    """(kernel, scratch bytes a lane, spilled vector registers) of every kernel
    in the compiler's report that has either, and the number of kernels in it.

    No kernel may: a vector register spilled ahead of the point where the lanes
    of a divergent block rejoin was lost for the other lanes, and pixels were
    wrong.  (Scalar registers spill to lanes of a vector register, whatever lanes
    are active.)"""
    bad, n = [], 0
    for part in re.split(r"remark:\s+Function Name: ", report)[1:]:
        n += 1
        scratch, spilled = (int(re.search(what + r"\D*: (\d+)", part).group(1))
                            for what in (r"ScratchSize \[bytes/lane\]", r"VGPRs Spill"))
        if scratch or spilled:
            bad.append((part.split()[0], scratch, spilled))
    return bad, n


def build(verbose: bool = False) -> str:
    objs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".o")
        cmd = [HIPCC] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
        if src.endswith(".cpp"):
            cmd[1:1] = ["-x", "hip"]
        if verbose:
            print(" ".join(cmd), flush=True)
        if src.endswith(".hip"):
            cmd[1:1] = REPORT
        r = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
        if r.returncode or verbose:
            print(r.stderr, file=sys.stderr, flush=True)
        else:  # without the report, and without the host pass's note on the feature flag
            print(*(x for x in r.stderr.splitlines() if "warning:" in x), sep="\n", end="", file=sys.stderr, flush=True)
        r.check_returncode()
        if src.endswith(".hip"):
            bad, n = spilling_kernels(r.stderr)
            if bad or n == 0:
                raise RuntimeError(f"{src}: kernels with spills or scratch memory: {bad}" if bad
                                   else f"{src}: no kernel in the compiler's report")
        objs.append(obj)
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    for o in objs:
        os.remove(o)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
