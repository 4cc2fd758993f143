"""Builds libfib.so (HIP, gfx950) in the package directory.

    python -m paper_2107_07104_amd.csrc.build

Every HIP source is compiled with packed FP32 arithmetic disabled
(-packed-fp32-ops); the host side of hipcc warns that it does not know that
target feature, which is harmless.

Paced kernels (FIB_PACED in fib_internal.h) get an `s_nop 0` after every
PACE vector instructions of a long basic block.  A wave that issues
an exp, log or rcp holds its SIMD to one vector instruction per 4.2 to 4.7
clocks for the next hundred or so, with any number of waves; an instruction
that leaves the vector pipe lets the SIMD go to another wave, and two waves or
more together then reach one per 3 clocks.  A wave alone on its SIMD only pays
for the s_nop (12 %).  Clocks of a Heun step of the 57-state model per SIMD,
and of 9 nodes of Hodgkin-Huxley:

    s_nop after every          none     3     4     5     6     7     8    12    16
    57 states, two waves       8033  6766  6532  6488  6446  6496  6529  6636  6739
    57 states, one wave        4497  5702  5374  5235  5054  5015  4943  4784  4695
    Hodgkin-Huxley, 2 waves     875   761   757   752   758   759   779   788   808

The s_nop cannot be put there from the source: the scheduler moves the vector
instructions past it, and most end up next to each other.  So a source with
paced kernels is compiled to assembly, spaced there, and assembled with the
tools beside the compiler; where one of those is missing or refuses its
arguments the source is compiled as it is, with a warning: the kernels are the
same, up to a fifth slower.  A paced kernel that does not come out spaced is an
error.
"""
from __future__ import annotations

import concurrent.futures
import os
import re
import subprocess
import sys
import tempfile
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.dirname(HERE)
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libfib.so")
SOURCES = ["fib_api.hip", "fib_kernels.hip", "mlp_api.hip", "mlp_kernels.hip",
           "surrogate_kernels.hip", "window_kernels.hip",
           "emg.hip", "probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
PACE = 6          # vector instructions between two s_nop
PACE_BLOCK = 48   # of a basic block that is spaced, at least
MARK = "; fib paced"

FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-munsafe-fp-atomics", "-Wall", "-Wno-unused-function", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"),
]

_PACED = re.compile(r"__global__[^;{]*?\b(k_\w+)\s*\([^{;]*\)\s*\{\s*FIB_PACED\(")


def llvm_dir() -> str:
    """The LLVM tools of the compiler in use, else of ROCM_PATH."""
    own = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(HIPCC))), "llvm", "bin")
    if os.path.isdir(own):
        return own
    return os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


_VALU = re.compile(r"\s+v_(?!nop)")
_OTHER = re.compile(r"\s+(s_|ds_|global_|buffer_|flat_|scratch_)")
_ENDS = re.compile(r"\s+s_(c?branch|endpgm|setpc|swappc)")


def _space(block: list[str]) -> list[str]:
    """A basic block's lines with an s_nop after every PACE vector
    instructions in a row.  Only lines that hold a vector instruction are
    followed by one, so pairs that the assembler reads together (s_getpc and
    the additions to it) stay together."""
    if sum(1 for l in block if _VALU.match(l)) < PACE_BLOCK:
        return block
    out, run = [], 0
    for line in block:
        out.append(line)
        if _VALU.match(line):
            run += 1
            if run == PACE:
                out.append("\ts_nop 0")
                run = 0
        elif _OTHER.match(line):
            run = 0
    return out


def pace(asm: str) -> tuple[str, int]:
    """The assembly with the functions that hold MARK spaced; and how many."""
    out, fn, n = [], [], 0

    def close():
        nonlocal n
        if not any(MARK in l for l in fn):
            out.extend(fn)
            return
        n += 1
        block = []
        for line in fn:
            label = line[:1] not in ("", "\t", " ", ";", "#") and ":" in line
            if label:
                out.extend(_space(block))
                block = []
            block.append(line)
            if _ENDS.match(line):
                out.extend(_space(block))
                block = []
        out.extend(_space(block))

    for line in asm.split("\n"):
        fn.append(line)
        if line.startswith(".Lfunc_end"):
            close()
            fn = []
    out.extend(fn)
    return "\n".join(out), n


def unspaced(src: str, asm: str) -> list[str]:
    """The kernels of a source that start with FIB_PACED but have no instance
    with an s_nop in the paced assembly."""
    spaced, fn = [], []
    for line in asm.split("\n"):
        fn.append(line)
        if line.startswith(".Lfunc_end"):
            if any(MARK in l for l in fn) and "\ts_nop 0" in fn:
                spaced += [l.split(":")[0] for l in fn if l[:1] not in ("", "\t", " ", ";", ".", "#")]
            fn = []
    return [k for k in _PACED.findall(src)
            if not any(f"{len(k)}{k}" in name or name == k for name in spaced)]


def _compile(src: str, obj: str, extra: list[str]) -> None:
    path = os.path.join(HERE, src)
    flags = [*FLAGS, *extra]

    def run(*cmd):
        subprocess.run(cmd, check=True)

    with open(path) as f:
        source = f.read()
    if "FIB_PACED" not in source:
        run(HIPCC, *flags, "-c", path, "-o", obj)
        return
    asm, dev, co, fatbin = (obj + e for e in (".s", ".dev.o", ".co", ".hipfb"))
    run(HIPCC, *flags, "--offload-device-only", "-S", path, "-o", asm)
    with open(asm) as f:
        text, n = pace(f.read())
    missing = unspaced(source, text)
    if not n or missing:
        raise RuntimeError(f"{src}: no paced instance in the assembly of {missing or 'any kernel'}")
    with open(asm, "w") as f:
        f.write(text)
    llvm = llvm_dir()
    try:
        run(os.path.join(llvm, "clang"), "-x", "assembler", "-target", "amdgcn-amd-amdhsa",
            f"-mcpu={ARCH}", "-c", asm, "-o", dev)
        run(os.path.join(llvm, "ld.lld"), "-shared", dev, "-o", co)
        run(os.path.join(llvm, "clang-offload-bundler"), "-type=o", "-bundle-align=4096",
            f"-targets=host-x86_64-unknown-linux-gnu,hipv4-amdgcn-amd-amdhsa--{ARCH}",
            "-input=/dev/null", f"-input={co}", f"-output={fatbin}")
        run(HIPCC, *flags, "--offload-host-only", "-Xclang", "-fcuda-include-gpubinary",
            "-Xclang", fatbin, "-c", path, "-o", obj)
    except (OSError, subprocess.CalledProcessError) as e:
        warnings.warn(f"{src}: built without spaced vector instructions ({e})", RuntimeWarning)
        run(HIPCC, *flags, "-c", path, "-o", obj)


def build(verbose: bool = False, extra=None) -> str:
    extra = list(extra or [])
    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as d:
        objs = [os.path.join(d, s + ".o") for s in SOURCES]
        with concurrent.futures.ThreadPoolExecutor(4) as pool:
            for s, job in [(s, pool.submit(_compile, s, o, extra))
                           for s, o in zip(SOURCES, objs)]:
                job.result()
                if verbose:
                    print(s, flush=True)
        subprocess.run([HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs],
                       check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
