"""Compiles the HIP library libselfjoin.so for gfx950 (in-tree)."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libselfjoin.so")
SOURCES = ["sj_api.hip", "sj_build.hip", "sj_refine.hip", "sj_lowp.hip", "sj_hits.hip", "sj_batch.hip", "sj_probe.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    # every rounding in the exact paths is explicit (fma / _rn intrinsics)
    "-ffp-contract=off",
    # no packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # MFMA accumulators in ordinary VGPRs (no AGPR copies around each tile)
    "-mllvm", "-amdgpu-mfma-vgpr-form",
]


def build(verbose: bool = False) -> str:
    """Compile every source (one hipcc each, side by side) and link them into
    libselfjoin.so; always recompiles."""
    tag = ".tmp%d" % os.getpid()
    tmp = LIB + tag
    objs = [os.path.join(CSRC, s + tag + ".o") for s in SOURCES]
    compile_flags = [f for f in FLAGS if f != "-shared"]
    try:
        runs = [subprocess.Popen([HIPCC] + compile_flags + ["-c", os.path.join(CSRC, s), "-o", o],
                                 stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
                for s, o in zip(SOURCES, objs)]
        outs = [r.communicate()[0] for r in runs]
        for s, r, text in zip(SOURCES, runs, outs):
            if r.returncode != 0:
                raise RuntimeError("hipcc failed on " + s + ":\n" + text)
        link = [HIPCC, "--offload-arch=gfx950", "-fPIC", "-shared"] + objs + ["-o", tmp]
        res = subprocess.run(link, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc link failed:\n" + res.stdout + res.stderr)
        if verbose:
            print("".join(outs) + res.stderr)
    finally:
        for o in objs:
            if os.path.exists(o):
                os.remove(o)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=False))
