"""Compile libqg.so (HIP kernels + C ABI) for gfx950 with hipcc, in place."""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libqg.so")
SOURCES = [os.path.join(CSRC, f) for f in ("qg_kernels.hip", "qg_graph.hip", "qg_api.cpp", "qg_graph.cpp",
                                            "qg_server.cpp")]
HEADERS = [os.path.join(CSRC, f) for f in ("qg_kernels.h", "qg_graph.h", "qg_layout.h", "qg_internal.h")] + [
    os.path.join(ROOT, "include", "qg.h")]

DIMS = (96, 128, 768, 960)  # the dimensions whose search kernels are built, one object each

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # every fused multiply-add is written out; division is IEEE correctly rounded
    "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt",
    # no packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def _run(cmd) -> str:
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed ({res.returncode}):\n{err}")
    return err


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    kernels = SOURCES[0]
    units = [(kernels, [f"-DQG_DIM={d}"]) for d in DIMS] + [(s, []) for s in SOURCES]
    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as obj:
        objects = [os.path.join(obj, f"{i}.o") for i in range(len(units))]
        cmds = [[hipcc] + FLAGS + defs + ["-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", src, "-o", o]
                for (src, defs), o in zip(units, objects)]
        with concurrent.futures.ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
            errs = list(pool.map(_run, cmds))
        errs.append(_run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objects + ["-o", tmp]))
    err = "\n".join(e for e in errs if e.strip())
    if verbose and err.strip():
        print(err, file=sys.stderr)
    os.replace(tmp, LIB)
    return LIB


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(s) > t for s in SOURCES + HEADERS)


if __name__ == "__main__":
    print(build(verbose=True))
