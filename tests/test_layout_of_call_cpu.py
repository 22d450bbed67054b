"""The layout of every call is a compiled one that holds the row, whatever the number of rows, and differs from the width's
own only where the rule for few wide rows says so."""
import os
import subprocess

from conftest import ROOT

PROGRAM = r"""
#include <stdio.h>
#include "rtopk_shape.hpp"
using namespace rtopk;
int main() {
  long bad = 0, other = 0;
  const int64_t counts[] = {1, 255, 256, 512, 513, 1024, 1025, 3072, 3073, 4096, 4097, 6144, 6145, 24576, 24577, 1 << 20, (int64_t)1 << 31};
  const int ks[] = {1, 99, 100, 256, 257, 512, 513, 700, 1000, 1025};
  for (int M = 1; M <= 70000; M += M < 9000 ? 1 : 37)
    for (int64_t N : counts)
      for (int k : ks)
        for (int dtype = 0; dtype < 3; ++dtype)
          for (int mode = 0; mode < (dtype == kF32 ? 3 : 2); ++mode)
            for (int dense = 0; dense < (dtype == kF32 && mode != kEps ? 2 : 1); ++dense)
              for (int steps = 4; steps < 9; steps += 4) {
                if (k > M || ((dtype != kF32 || dense) && M > kMaxBlockM)) continue;
                const bool plain = dtype == kF32 && mode != kEps;
                const Shape a = kernel_layout(M, dtype, plain, dense), b = layout_of_call(N, M, k, dtype, mode, steps, plain, dense);
                const bool same = a.family == b.family && a.g == b.g && a.ng == b.ng && a.w == b.w && a.full == b.full;
                if (!instantiated(b, dtype, plain, dense) || (b.family != kFamStream && b.capacity() < M)) ++bad;
                if (b.full != (b.g != 0 && b.family != kFamStream && M == b.capacity())) ++bad;
                if (same) continue;
                const bool lists = M > 1536 && M <= kMaxWaveM && k <= filter_max_k(4) && b.w == 4 && (mode != kEarly || steps >= 5);
                const bool longer = mode == kExact && !dense && M > 2048 && M <= 16384 && k > filter_max_k(4) &&
                                    k <= big_filter_max_k(b.w) && (b.w == 4 || b.w == 8);
                if (k == M || N >= 0x80000000ll || !(lists || longer)) ++bad;
                ++other;
              }
  printf("%ld %ld\n", bad, other);
  return 0;
}
"""


def test_layout_of_every_call(tmp_path):
    src = tmp_path / "layouts.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "layouts"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "paper_2409_00822_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    bad, other = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert bad == 0 and other > 0
