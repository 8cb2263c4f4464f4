"""Host code of the device headers and the block-level logic of small kernels,
compiled for the CPU against a stand-in for the HIP headers (hostsim/)."""
import glob
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = os.path.join(os.path.dirname(os.path.realpath(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"))),
                   "..", "llvm", "bin", "clang++")
FLAGS = ["-std=c++17", "-O1", "-pthread", "-Wno-unknown-pragmas", "-fsanitize=undefined",
         "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "tests", "hostsim")]


def _run(tmp_path, source):
    if not os.path.exists(CXX):
        pytest.skip("no host compiler of the ROCm toolchain")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(source)
    for h in glob.glob(os.path.join(ROOT, "paper_2001_10424_amd", "csrc", "*.hpp")):
        # block-shared variables are static here, those of dynamic size external
        with open(h) as f:
            (tmp_path / os.path.basename(h)).write_text(f.read().replace("extern __shared__", "extern"))
    res = subprocess.run([CXX, *FLAGS, "-I", str(tmp_path), str(src), "-o", str(exe)],
                         capture_output=True, text=True)
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


# a block of 256 threads of which waves 2 and 3 start after waves 0 and 1 wait
# at their first barrier and `meanwhile` has run
BLOCK = r"""
#include <cstdio>
#include <functional>
#include <thread>
#include <vector>
#include "fgmres.hpp"
using namespace gkb;
void run_block(int block, int blocks, std::function<void()> kernel, std::function<void()> meanwhile) {
  gridDim = dim3(blocks);
  hostsim::block.reset(256);
  for (int w = 0; w < 4; ++w) hostsim::wave[w].reset(64);
  std::vector<std::thread> t;
  auto start = [&](int first) {
    for (int i = first; i < first + 128; ++i)
      t.emplace_back([=] {
        threadIdx = dim3(i, 0, 0), blockIdx = dim3(block, 0, 0);
        kernel();
        hostsim::block.leave();
      });
  };
  start(0);
  while (hostsim::block.stopped() < 128) std::this_thread::yield();
  meanwhile();
  start(128);
  for (auto& x : t) x.join();
}
"""


def test_update_of_a_block_that_starts_while_the_solve_ends(tmp_path):
    """The folded PCG update meets p.q <= 0: block 0 ends the solve, and a
    block leaves x and r as they are, whether its waves read the flag before
    and after that or all before, also where the direction is not finite."""
    _run(tmp_path, BLOCK + r"""
int main() {
  const int n = 512;
  std::vector<double> x(n, 3.0), r(n, 5.0), p(n, 1.0), q(n, 1.0), part(256), rr(2, -1.0);
  for (int i = 0; i < 256; ++i) part[i] = i < 128 ? 1.0 : -2.0;  // the sum is negative
  p[300] = q[310] = NAN;
  PcgState st{};
  st.rz = 1.0;
  for (int flag : {1, 0}) {
    st.done = 0;
    run_block(1, 2, [&] { k_pcg_xr_fold<double>(n, &st, part.data(), 256, p.data(), q.data(),
                                                x.data(), r.data(), rr.data()); },
              [&] { st.done = flag; });
    for (int i = 0; i < n; ++i)
      if (x[i] != 3.0 || r[i] != 5.0) return std::printf("entry %d: %g %g\n", i, x[i], r[i]), 1;
  }
  return 0;
}
""")


def test_basis_vector_of_a_block_that_starts_while_the_cycle_ends(tmp_path):
    """The next basis vector where block 0 ends the cycle: a late block writes
    its part with the right norm or not at all."""
    _run(tmp_path, BLOCK + r"""
int main() {
  const int n = 512;
  std::vector<double> w(n, 6.0), v(n, -1.0), part(256, 1.0 / 64);  // ||w||^2 = 4
  static FgmState fs;
  PcgState st{}, cyc{};
  run_block(1, 2, [&] { k_gm_next<double>(n, &st, &cyc, &fs, part.data(), 256, 1, w.data(), v.data(),
                                          nullptr, nullptr, CsrOps<double>{}, nullptr); },
            [&] { cyc.done = 1; });
  for (int i = 256; i < n; ++i)
    if (v[i] != v[256] || (v[i] != -1.0 && v[i] != 3.0)) return std::printf("%d %g\n", i, v[i]), 1;
  return 0;
}
""")
