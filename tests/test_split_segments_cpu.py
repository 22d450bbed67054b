"""Which rows of more than 32768 columns are cut into segments of 16384 columns instead of 32768 when there are rows enough to fill the
GPU with either: not with many rows where the longer ones fill their lanes or lists are long, which made those calls up to 15 % slower."""
import os
import subprocess

import pytest

from conftest import ROOT

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "rtopk_shape.hpp"
using namespace rtopk;
int main(int argc, char** argv) {
  for (int i = 1; i + 3 < argc; i += 4) {
    const int steps = atoi(argv[i + 3]);
    printf("%d ", split_of(atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]), steps ? kEarly : kExact, steps).w);
  }
  return 0;
}
"""

# (rows, columns, k, steps of early stopping or 0: exact mode), on both sides of each line
LONG = [(356, 34424, 250, 0), (700, 59000, 150, 0), (1000, 65536, 8, 0), (700, 65536, 64, 8), (334, 98304, 16, 0), (500, 131072, 100, 0), (256, 196608, 8, 0),
        (430, 65535, 64, 0), (700, 49152, 8, 0), (367, 70000, 8, 16), (500, 70001, 134, 0), (1000, 50000, 134, 0), (2048, 50000, 100, 0),
        (320, 50000, 200, 0), (640, 50001, 200, 0), (300, 62000, 250, 0), (320, 62000, 200, 0), (640, 62000, 160, 0), (768, 62000, 100, 0), (768, 62001, 134, 0),
        (330, 128000, 48, 0), (360, 127999, 48, 0), (600, 41000, 161, 0), (128, 262144, 48, 4), (512, 131072, 8, 4)]
SHORT = [(360, 33000, 8, 0), (700, 36000, 128, 0), (360, 50000, 128, 0), (1023, 50000, 32, 0), (767, 50000, 64, 0), (700, 62000, 16, 0), (300, 80000, 64, 0),
         (300, 94000, 33, 0), (300, 110000, 100, 0), (400, 126000, 8, 0), (120, 164776, 55, 0), (100, 230000, 64, 0), (1, 65536, 256, 0), (64, 131072, 50, 0),
         (310, 65536, 48, 0), (420, 65535, 64, 0), (550, 44000, 64, 0), (550, 44000, 134, 0), (500, 70001, 100, 0), (800, 50000, 134, 0), (300, 50000, 200, 0),
         (600, 50001, 200, 0), (300, 62000, 200, 0), (600, 62000, 160, 0), (767, 62000, 100, 0), (767, 62001, 134, 0), (310, 128000, 48, 0), (350, 127999, 48, 0),
         (127, 262144, 48, 4), (511, 131072, 8, 4), (217, 112484, 134, 4)]


@pytest.mark.parametrize("cases, wavefronts", [(LONG, 8), (SHORT, 4)])
def test_wavefronts_of_a_segment(tmp_path, cases, wavefronts):
    src = tmp_path / "segments.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "segments"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "paper_2409_00822_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    args = [str(v) for case in cases for v in case]
    got = list(map(int, subprocess.run([str(exe)] + args, check=True, capture_output=True, text=True).stdout.split()))
    wrong = [case for case, w in zip(cases, got) if w != wavefronts]
    assert len(got) == len(cases) and not wrong, wrong
