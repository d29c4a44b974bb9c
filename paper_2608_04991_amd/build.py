"""Build the gfx950 HIP library (librac.so) in-tree with hipcc.

Flags: -ffp-contract=off keeps every multiply and add separately rounded (the
codec's arithmetic is defined operation by operation); packed fp32 ops are
disabled; divisions stay correctly rounded (hipcc's default).

The device assembly is also generated and scanned for a known miscompile
(see isa_check.py); a hit fails the build.
"""
from __future__ import annotations

import os
import subprocess
import sys

try:
    from . import isa_check
except ImportError:  # run as a script
    import isa_check

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "csrc", "rac.hip")
HOST_SRC = os.path.join(HERE, "csrc", "spans.cpp")   # host-only C++ (reference selection)
PRED_SRC = os.path.join(HERE, "csrc", "predictor.hip")  # decode-phase reference predictor
INC = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "lib", "librac.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-ffp-contract=off", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


PARTS = (None, 2, 3, 4, 8)  # rac.hip: everything but the per-width kernels, then one bit width each


def build(verbose: bool = True) -> str:
    out = os.path.dirname(LIB)
    os.makedirs(out, exist_ok=True)
    compile_flags = [f for f in FLAGS if f != "-shared"]
    # every object, and the device assembly of the codec's parts that is
    # scanned, are independent compiles: run them side by side
    jobs, objs, asms = [], [], []
    for part in PARTS:
        define = [] if part is None else [f"-DRAC_PART={part}"]
        name = os.path.join(out, f"rac_{part or 'main'}")
        objs.append(name + ".o")
        asms.append(name + ".s")
        jobs.append([HIPCC, *compile_flags, *define, "-c", "-I", INC, "-o", objs[-1], SRC])
        jobs.append([HIPCC, *[f for f in compile_flags if f != "-fPIC"], *define, "--cuda-device-only", "-S",
                     "-I", INC, "-o", asms[-1], SRC])
    for src in (PRED_SRC, HOST_SRC):
        objs.append(os.path.join(out, os.path.basename(src) + ".o"))
        jobs.append([HIPCC, *compile_flags, "-c", "-I", INC, "-o", objs[-1], src])
    tmp = LIB + ".tmp"
    try:
        if verbose:
            for cmd in jobs:
                print(" ".join(cmd), flush=True)
        procs = [subprocess.Popen(cmd) for cmd in jobs]
        codes = [p.wait() for p in procs]
        for code, cmd in zip(codes, jobs):
            if code:
                raise subprocess.CalledProcessError(code, cmd)
        bad = [hit for asm in asms for hit in isa_check.scan(open(asm).read())]
        if bad:
            raise RuntimeError("miscompiled SCC use in librac:\n" + "\n".join(bad))
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], check=True)
        os.replace(tmp, LIB)
    finally:
        for f in (tmp, *objs, *asms):
            if os.path.exists(f):
                os.remove(f)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
