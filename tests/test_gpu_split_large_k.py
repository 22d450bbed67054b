"""GPU parity of split rows with large k: lists of up to 1792 candidates from segments of 32768 or 65536 columns, merges of up to 40
candidates per lane, segments that crowd, k on both sides of the limits; and the layout of every split, on the CPU.

Selections are copies of inputs and their columns: tolerance 0.
"""
import os
import subprocess

import numpy as np
import pytest

import oracle
from conftest import ROOT
from test_gpu_filtered_rows import _gpu, _rows, _same
from test_gpu_list_bins import _bins_rows

torch = pytest.importorskip("torch")


def _large_rows(M, k, seed):
    g = np.random.default_rng(seed)
    x = np.concatenate([_rows(M, seed)[:4], _bins_rows(M, k, seed)[[0, 2, 7, 8, 10, 13]]])
    x = np.concatenate([x, np.sort(x[:1], axis=1), np.sort(x[:1], axis=1)[:, ::-1], g.integers(0, 50, (2, M)).astype(np.float32)])
    crowd = g.standard_normal((1, M)).astype(np.float32)
    crowd[0, : 3 * k] += 20  # the winners in one segment
    return np.concatenate([x, crowd]).astype(np.float32)


@pytest.mark.gpu
@pytest.mark.parametrize("M, k", [(65537, 513), (65537, 1024), (70001, 1000), (131075, 600), (131072, 1024), (300000, 1024),
                                  (330001, 1024), (700001, 513), (700001, 1000), (1 << 20, 300), (1 << 20, 700), (1 << 20, 1024),
                                  (131075, 1025)])
def test_every_mode(M, k):
    R = _gpu()
    x = _large_rows(M, k, M + k)
    xd = torch.from_numpy(x).cuda()
    tag = f"M={M} k={k}"
    _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(x, k), tag + " exact")
    _same(R.rtopk_rowwise_exact_smallest(xd, k), oracle.topk_exact_smallest(x, k), tag + " smallest")
    for mi in (8, 40):
        _same(R.rtopk_rowwise(xd, k, mi), oracle.topk_earlystop(x, k, mi), tag + f" early {mi}")
    for eps in (0.05, 1e-5):
        ev, ei, et = oracle.alg1(x, k, eps_rel=eps)
        got = R.rtopk_rowwise_eps(xd, k, eps, want_iters=True)
        _same(got, (ev, ei), tag + f" eps {eps}")
        assert np.array_equal(got[2].cpu().numpy(), et), tag + " iterations"


PROGRAM = r"""
#include <stdio.h>
#include <initializer_list>
#include "rtopk_shape.hpp"
using namespace rtopk;
int main() {
  long bad = 0, split = 0;
  for (int64_t M = 32769; M <= kMaxM; M += M < 66000 ? 7 : M / 67 + 1)
    for (int k = 1; k <= 1100; k += k < 20 ? 1 : 17)
      for (int64_t N : {(int64_t)1, (int64_t)64, (int64_t)100000})
        for (int call = 0; call < 9; ++call) {
          static const int steps_of[] = {8, 0, 1, 2, 4, 5, 7};
          const int mode = call < 7 ? (int)kEarly : (call == 7 ? (int)kExact : (int)kEps), steps = call < 7 ? steps_of[call] : 0;
          const Split s = split_big_of(N, (int)M, k, mode, steps);
          if (mode == kEarly && s.segments != 0 && !splits_early(N, (int)M, steps)) ++bad;
          if (s.segments == 0) continue;
          ++split;
          const int64_t last = M - (int64_t)(s.segments - 1) * s.length;
          const bool ok = M > kMaxBlockM && k <= kBigMaxK && s.big && (s.w == 8 || s.w == 16) && s.ng == 16 && s.merge_waves == 16 &&
                          s.segments >= 2 && s.segments <= kMaxSegments && s.length % 4 == 0 && s.length <= 64 * s.w * 4 * s.ng &&
                          last > 0 && last <= s.length && s.cap > k && s.cap <= kBigRoom &&
                          (int64_t)s.segments * s.cap <= 16 * 64 * kMergeRegsBig && s.rows >= 1 && s.rows <= N &&
                          s.rows * s.segments <= 0x7fffffff && (s.rows == 1 || s.bytes() <= kSplitScratch) &&
                          // every wavefront has maxima of eight values for its share of the floor
                          (last / (64 * s.w * 4)) / 2 * 64 >= (k + s.w) / s.w;
          if (!ok) ++bad;
        }
  printf("%ld %ld\n", bad, split);
  return 0;
}
"""


def test_every_split_fits_its_lists_and_the_merge(tmp_path):
    src = tmp_path / "splits.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "splits"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "paper_2409_00822_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    bad, split = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert bad == 0 and split > 0
