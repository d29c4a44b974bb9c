"""What a call would launch, seen without a GPU: the calls run in a child
process in which tests/hip_recorder.cpp stands in for the HIP runtime."""
from __future__ import annotations

import json
import os
import re
import subprocess
import sys
from typing import NamedTuple

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_CHILD = r"""
import ctypes, json, sys
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rec.recorded.restype = rec.registered.restype = ctypes.c_char_p
import paper_2608_04991_amd as rac
P = 1 << 20  # a stand-in for every device pointer (aligned; nothing reads it)
out = []
for kind, arg in json.load(sys.stdin):
    rec.forget()
    if kind == "all":
        rac.library()
        out.append(rec.registered().decode())
        continue
    if kind == "predictor":
        *cfg, batch = arg
        c = rac.PredictorConfig(*cfg)
        rac.rac_predictor_step(c, P, P, P, P, P, P, batch, 0)
    elif kind == "calibrate":
        cs = [rac.RacConfig(*c) for c in arg]
        rac.rac_calibrate(P, P, cs, 1e-3, P, 0)
    else:
        c = rac.RacConfig(*arg)
        n = rac.rac_wire_size(c)
        if kind in ("encode", "encode_zero"):
            rac.rac_encode(c, P, P if kind == "encode" else None, P if c.flags & 1 else None, P, P, 0, n)
        elif kind == "pooled":
            rac.rac_encode_pooled(c, P, P, P, None, P, P, 0, segments=5, wire_cap=n)
        elif kind == "decode":
            rac.rac_decode(c, P, P, P if c.flags & 1 else None, P, 0)
    out.append(rec.recorded().decode())
print(json.dumps(out))
"""


class Launch(NamedTuple):
    kernel: str  # e.g. "pred_prod<1, 4, 4, 2, 1, true, 16>"
    grid: int
    grid_y: int
    threads: int
    lds: int


def launches(calls, tmp) -> list[list[Launch]]:
    """The launches of each call: ("encode" | "encode_zero" (no reference) |
    "decode" | "pooled", RacConfig fields), ("predictor", PredictorConfig fields + [batch]) or ("calibrate",
    list of RacConfig fields).  ("all", None) gives every kernel of the library."""
    so = os.path.join(str(tmp), "hip_recorder.so")
    if not os.path.exists(so):
        subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(ROOT, "tests", "hip_recorder.cpp")],
                       check=True)
    r = subprocess.run([sys.executable, "-c", _CHILD, so], cwd=ROOT, input=json.dumps(calls), text=True,
                       stdout=subprocess.PIPE, check=True, timeout=300)
    logs = json.loads(r.stdout)
    mangled = sorted({l.split("\t")[0] for log in logs for l in log.splitlines()})
    plain = subprocess.run(["c++filt"], input="\n".join(mangled), text=True, capture_output=True,
                           check=True).stdout.splitlines()
    name = {m: re.sub(r"\(anonymous namespace\)::|^void ", "", p).split("(")[0] for m, p in zip(mangled, plain)}
    return [[Launch(name[f[0]], *map(int, f[1:])) for f in (l.split("\t") for l in log.splitlines())] for log in logs]
