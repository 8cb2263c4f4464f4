"""Host code of the device headers and the block-level logic of small kernels,
compiled for the CPU against a stand-in for the HIP headers (hostsim/)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = os.path.join(os.path.dirname(os.path.realpath(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"))),
                   "..", "llvm", "bin", "clang++")
FLAGS = ["-std=c++17", "-O1", "-pthread", "-Wno-unknown-pragmas", "-fsanitize=undefined",
         "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "tests", "hostsim"),
         "-I", os.path.join(ROOT, "paper_2001_10424_amd", "csrc")]


def _run(tmp_path, source):
    if not os.path.exists(CXX):
        pytest.skip("no host compiler of the ROCm toolchain")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(source)
    res = subprocess.run([CXX, *FLAGS, str(src), "-o", str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, (res.returncode, res.stdout[-2000:], res.stderr[-2000:])


def test_march_chunks_of_any_depth(tmp_path):
    """Every depth from the two planes that a grid may have gets chunks of an
    even number of planes, at least four, that cover it without an empty one
    (but for grids shallower than a chunk)."""
    _run(tmp_path, r'''
#include <cstdio>
#include "legs.hpp"
int main() {
  for (int columns : {1, 7, 64, 128, 255, 256, 1024, 65536})
    for (int nz = 1; nz <= 300; ++nz) {
      const int tz = gkb::march_planes(columns, nz), chunks = (nz + tz - 1) / tz;
      if (tz < 4 || tz % 2 || chunks < 1 || (chunks - 1) * tz >= nz) {
        std::printf("columns %d nz %d tz %d\n", columns, nz, tz);
        return 1;
      }
    }
  return 0;
}
''')
