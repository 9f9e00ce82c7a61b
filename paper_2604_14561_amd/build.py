"""Build libcocodiff.so (hand-written HIP for gfx950) in-tree with hipcc, and the binding's native part with gcc."""
from __future__ import annotations

import glob
import os
import re
import subprocess
import sysconfig
import tempfile
import warnings
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libcocodiff.so")
# the binding's native part, for this interpreter
MARSHAL_SOURCE = os.path.join(_HERE, "csrc", "marshal.c")
MARSHAL_PATH = os.path.join(_HERE, "_marshal" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
SOURCES = sorted(glob.glob(os.path.join(_HERE, "csrc", "*.hip")))

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc", "-fvisibility=hidden",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # a kernel's leading plain arguments, up to the first structure, arrive in registers (no wait for the memory that holds
    # them): all of the token metric's, top-k's and the copy's, the pointers of the permutations and the list moves.  (Whole
    # calls without and with it: a cache update by tokens 131.2 and 127.8 us, by tiles 57.0 and 55.8, nothing elsewhere)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-inline-asm",
]


def _run(cmd: list) -> str:
    proc = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 feature and says so; that is harmless
    err = "\n".join(l for l in proc.stderr.splitlines() if "packed-fp32-ops" not in l)
    if proc.returncode != 0:
        raise RuntimeError(os.path.basename(cmd[0]) + " failed:\n" + err)
    return err


def accumulator_accesses(assembly: str) -> list:
    """Instructions of the projection's main kernels (device assembly of gemm_*.hip) that touch an accumulation register
    outside inline assembly.  Those kernels keep their accumulators in a0 .. by number, unknown to the compiler; nothing in the
    language forbids it a short-lived copy there, so what it made is looked at: (line number, instruction) of each."""
    found, kernel, inline = [], False, False
    for n, line in enumerate(assembly.splitlines(), 1):
        if re.match(r"[A-Za-z_]\w*:", line):
            kernel = "qkv_gemm_direct_kernel" in line
        elif "#ASMSTART" in line:
            inline = True
        elif "#ASMEND" in line:
            inline = False
        elif kernel and not inline and re.match(r"\t[a-z]", line):
            instruction = line.split(";")[0].strip()
            if re.search(r"[\s,\[]a(\d+\b|\[)", instruction):
                found.append((n, instruction))
    return found


def scratch_users(assembly: str) -> list:
    """(kernel, bytes per lane) of the projection's main kernels that spill vector registers to scratch memory."""
    sizes = re.findall(r"\.name:\s+(\S*qkv_gemm_direct_kernel\S*)\s+\.private_segment_fixed_size:\s+(\d+)", assembly)
    return [(name, int(size)) for name, size in sizes if int(size)]


def _check_assembly(source: str, obj: str) -> None:
    path = obj[:-len(".hip.o")] + "-hip-amdgcn-amd-amdhsa-gfx950.s"
    with open(path) as f:
        assembly = f.read()
    if "qkv_gemm_direct_kernel" in assembly:
        found = accumulator_accesses(assembly)
        if found:
            raise RuntimeError(f"{os.path.basename(source)}: the compiler uses accumulation registers of its own in "
                               f"{len(found)} instructions, the first {found[0][1]!r}: they hold the projection's accumulators")
        spilled = scratch_users(assembly)
        if spilled:
            raise RuntimeError(f"{os.path.basename(source)}: {len(spilled)} kernels spill registers, the first {spilled[0]}")


def _compile(cmd: list) -> str:
    err = _run(cmd)
    _check_assembly(cmd[-3], cmd[-1])
    return err


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    jobs = min(len(SOURCES), int(os.environ.get("MAX_JOBS", "0")) or os.cpu_count() or 1, 8)
    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(jobs) as pool:
        objects = [os.path.join(tmp, os.path.basename(s) + ".o") for s in SOURCES]
        cmds = [[hipcc] + HIPCC_FLAGS + ["-save-temps=obj", "-c", s, "-o", o] for s, o in zip(SOURCES, objects)]
        cmds[:] = sorted(cmds, key=lambda c: "gemm_fused" not in c[-3])      # the longest first
        for err in pool.map(_compile, cmds):
            if verbose and err.strip():
                print(err)
        _run([hipcc] + HIPCC_FLAGS + ["-shared", "-o", LIB_PATH] + objects)
    include = sysconfig.get_paths()["include"]
    if os.path.exists(os.path.join(include, "Python.h")):
        _run([os.environ.get("CC", "gcc"), "-O2", "-std=gnu11", "-Wall", "-shared", "-fPIC", "-I", include, MARSHAL_SOURCE, "-o", MARSHAL_PATH])
    else:      # the library needs no Python, and the binding works without its native part
        if os.path.exists(MARSHAL_PATH):
            os.remove(MARSHAL_PATH)
        warnings.warn(f"no Python.h in {include}: the binding's native part is not built, and calls take the host longer", RuntimeWarning)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
