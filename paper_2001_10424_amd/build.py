"""Compile the HIP sources of the package into the in-tree shared library
``libgkb.so`` for gfx950 (hipcc cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgkb.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


SOURCES = ("gkb.hip", "legs.hip", "march.hip", "conv.hip")


def sources():
    return [os.path.join(CSRC, f) for f in SOURCES]


def build_library(verbose: bool = False) -> str:
    """Every source to an object (in parallel), then the shared library."""
    inc = ["-I", os.path.join(ROOT, "include")]
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, os.path.basename(f) + ".o") for f in sources()]
        jobs = [subprocess.Popen([HIPCC, *FLAGS, *inc, "-c", src, "-o", obj],
                                 stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
                for src, obj in zip(sources(), objs)]
        logs = [j.communicate()[0] for j in jobs]
        failed = [log for j, log in zip(jobs, logs) if j.returncode != 0]
        if failed:
            raise RuntimeError("hipcc failed:\n" + failed[0][-8000:])
        out = LIB + ".tmp"
        res = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-o", out, *objs],
                             capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + res.stderr[-8000:])
        if verbose and "".join(logs):
            print("".join(logs)[-2000:])
        os.replace(out, LIB)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
