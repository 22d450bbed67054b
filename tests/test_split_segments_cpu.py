"""Which rows of more than 32768 columns are cut into segments of 16384 columns instead of 32768 when there are rows enough to fill the
GPU with either: not where the longer ones fill their lanes, nor with long lists, which made those calls up to 11 % slower."""
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
  for (int i = 1; i + 2 < argc; i += 3) printf("%d ", split_of(atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]), kExact, 0).w);
  return 0;
}
"""

LONG = [(356, 34424, 250), (700, 59000, 150), (1000, 65536, 8), (700, 65536, 64), (334, 98304, 16), (500, 131072, 100), (256, 196608, 8),
        (700, 49152, 8), (550, 44000, 64), (367, 70000, 8), (1000, 50000, 100), (2048, 50000, 100)]
SHORT = [(360, 33000, 8), (700, 36000, 128), (360, 50000, 128), (1023, 50000, 32), (767, 50000, 64), (700, 62000, 16), (300, 80000, 64),
         (300, 94000, 33), (300, 110000, 100), (400, 126000, 8), (120, 164776, 55), (100, 230000, 64), (1, 65536, 256), (64, 131072, 50)]


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
