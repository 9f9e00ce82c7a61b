"""Build libcocodiff.so (hand-written HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import glob
import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libcocodiff.so")
SOURCES = sorted(glob.glob(os.path.join(_HERE, "csrc", "*.hip")))

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc", "-fvisibility=hidden",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-inline-asm",
]


def _run(cmd: list) -> str:
    proc = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 feature and says so; that is harmless
    err = "\n".join(l for l in proc.stderr.splitlines() if "packed-fp32-ops" not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    return err


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    jobs = min(len(SOURCES), int(os.environ.get("MAX_JOBS", "0")) or os.cpu_count() or 1, 8)
    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(jobs) as pool:
        objects = [os.path.join(tmp, os.path.basename(s) + ".o") for s in SOURCES]
        cmds = [[hipcc] + HIPCC_FLAGS + ["-c", s, "-o", o] for s, o in zip(SOURCES, objects)]
        cmds[:] = sorted(cmds, key=lambda c: "gemm_fused" not in c[-3])      # the longest first
        for err in pool.map(_run, cmds):
            if verbose and err.strip():
                print(err)
        _run([hipcc] + HIPCC_FLAGS + ["-shared", "-o", LIB_PATH] + objects)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
