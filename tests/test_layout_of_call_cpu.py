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
                const Shape a = kernel_layout(M, dtype), b = layout_of_call(N, M, k, dtype, mode, steps, dense);
                const bool same = a.family == b.family && a.g == b.g && a.ng == b.ng && a.w == b.w && a.full == b.full;
                if (!instantiated(b, dtype, dense) || (b.family != kFamStream && b.capacity() < M)) ++bad;
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


SEARCHES = r"""
#include <initializer_list>
#include <stdio.h>
#include "rtopk_shape.hpp"
using namespace rtopk;
int main() {
  long bad = 0, unreached = 0, kernels = 0;
  // by 16 bits, mode, dense form, values per lane / 4, wavefronts
  static int asked[2][3][2][17][17];
  for (int M = 1; M <= kMaxBlockM; M += M < 8200 ? (M > 4080 && M < 4110 ? 1 : 23) : 1 + M / 50)
    for (int64_t N = 1; N <= 100000; N = N < 512 ? 512 : (N == 512 ? 4096 : N * 25))
      for (int k = 1; k <= 1200 && k <= M; k += 17)
        for (int half = 0; half < 2; ++half)
          for (int mode = 0; mode < (half ? 2 : 3); ++mode)
            for (int form = 0; form < (half || mode == kEps ? 1 : 2); ++form)  // pairs, dense
              for (int steps = 4; steps < 9; steps += 4) {
                const bool dense = form == 1;
                const int dtype = half ? kBF16 : kF32;
                const Shape s = layout_of_call(N, M, k, dtype, mode, steps, dense);
                if (s.family != kFamBlock) continue;
                for (float eps : {0.0f, 1e-6f, 1e-2f}) {
                  const int search = block_search(s, M, k, dtype, mode, steps, dense, N, eps);
                  asked[half][mode][dense][s.values() / 4][s.w] |= search;
                  if ((block_kernels(s.values(), s.w, mode, dense, half) & search) == 0) ++bad;
                }
              }
  for (int half = 0; half < 2; ++half)
    for (int mode = 0; mode < 3; ++mode)
      for (int dense = 0; dense < 2; ++dense)
        for (int e = 0; e < 17; ++e)
          for (int w = 0; w < 17; ++w) {
            Shape s{};
            s.family = kFamBlock;
            s.g = half ? 8 : 4;
            s.ng = 4 * e / s.g;
            s.w = w;
            const int dtype = half ? kBF16 : kF32;
            if ((half && (dense || mode == kEps || e % 2)) || (dense && mode == kEps)) continue;
            if (!instantiated(s, dtype, dense)) continue;
            const int compiled = block_kernels(4 * e, w, mode, dense, half);
            for (int bit = 1; bit < 8; bit <<= 1) {
              kernels += (compiled & bit) != 0;
              unreached += (compiled & bit) != 0 && (asked[half][mode][dense][e][w] & bit) == 0;
              if ((compiled & bit) != 0 && (asked[half][mode][dense][e][w] & bit) == 0)
                fprintf(stderr, "half %d mode %d dense %d values %d w %d search %d\n", half, mode, dense, 4 * e, w, bit);
            }
          }
  printf("%ld %ld %ld\n", bad, unreached, kernels);
  return 0;
}
"""


def test_the_compiled_searches_of_a_workgroup_are_those_that_calls_ask_for(tmp_path):
    src = tmp_path / "searches.cpp"
    src.write_text(SEARCHES)
    exe = tmp_path / "searches"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "paper_2409_00822_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    bad, unreached, kernels = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert bad == 0 and unreached == 0 and kernels > 0
