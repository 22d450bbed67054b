"""A workgroup that takes the lists of candidates has the group maxima for them: every wavefront's share of the row's floor is
well below the maxima it has, counted load by load from the layout, and the candidates expected above such a floor fit the
list.  (Results are the same where they do not fit: the search over the row runs behind the lists then, and only time shows it.)"""
import os
import subprocess

from conftest import ROOT

PROGRAM = r"""
#include <initializer_list>
#include <math.h>
#include <stdio.h>
#include <string.h>
#include "rtopk_shape.hpp"
using namespace rtopk;
int main() {
  long bad = 0, lists = 0, longer = 0, rows = 0;
  for (int M = 1; M <= kMaxBlockM; M += M < 8400 ? (M < 1500 ? 499 : 17) : 611)
    for (int64_t N : {(int64_t)64, (int64_t)512, (int64_t)4096, (int64_t)100000})
      for (int k = 1; k <= 1100 && k <= M; k += k < 40 ? 13 : 31)
        for (int dtype : {(int)kF32, (int)kBF16})
          for (int mode = 0; mode < (dtype == kF32 ? 3 : 2); ++mode)
            for (int form = 0; form < (dtype == kF32 ? 2 : 1); ++form) {  // pairs, and the dense form or a small precision
              const bool dense = form == 1 && mode != kEps;
              const float eps = form == 1 ? 1e-6f : 1e-2f;
              const Shape s = layout_of_call(N, M, k, dtype, mode, 8, dense);
              if (s.family != kFamBlock) continue;
              const int search = block_search(s, M, k, dtype, mode, 8, dense, N, eps), E = s.values();
              // as many values per lane as fill twelve loads or more: the lists wherever k is within their limit
              if (E >= 48 && (search == kSearchLists) != (k <= filter_max_k(s.w))) ++bad;
              if (search == kSearchRow) {
                ++rows;
                continue;
              }
              const bool big = search == kSearchLongLists;
              (big ? longer : lists) += 1;
              const int group = E / floor_groups(E, big), room = big ? big_list_room(s.w) : list_room(s.w);
              // wavefront by wavefront: its loads, and the groups of its lanes that hold a column
              static char seen[16][64][64];
              int maxima[16] = {}, loads[16] = {}, total = 0;
              memset(seen, 0, sizeof(seen));
              for (int i = 0; i * s.g < M; ++i) {
                const int wave = i / 64 % s.w, round = i / (64 * s.w);
                ++loads[wave];
                for (int e = round * s.g; e < (round + 1) * s.g; e += group < s.g ? group : s.g) {
                  char& at = seen[wave][i % 64][e / group];
                  maxima[wave] += at ? 0 : 1;
                  at = 1;
                }
              }
              for (int w = 0; w < s.w; ++w) {
                const int share = floor_share(M, s.g, s.w, w, floor_shares(M, k, s.g));
                if (loads_before(M, s.g, s.w, w + 1) - loads_before(M, s.g, s.w, w) != loads[w] || loads[w] < 64) ++bad;
                const double part = share / (double)maxima[w];
                if (part > 0.75 || M * (1 - pow(1 - part, 1.0 / group)) > 0.75 * room) ++bad;
                total += share;
              }
              if (total < k + 1 || total > (k + 1 > s.w ? k + 1 : k + s.w)) ++bad;
            }
  printf("%ld %ld %ld %ld\n", bad, lists, longer, rows);
  return 0;
}
"""


def test_every_list_has_the_maxima_for_its_floor(tmp_path):
    src = tmp_path / "lists.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "lists"
    subprocess.run(["g++", "-std=c++17", "-O2", "-I" + os.path.join(ROOT, "paper_2409_00822_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    bad, lists, longer, rows = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert bad == 0 and lists > 0 and longer > 0 and rows > 0, (bad, lists, longer, rows)
