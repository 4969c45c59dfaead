"""The LDS places of the image-quality kernel (host check, no GPU): every
column sum is written and read inside its row of the array, and the outputs
that are kept read exactly the columns of their windows."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_05643_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "ug_quality_tile.h"
using namespace ug;
int main() {
  int column[kQPitch], bad = 0;
  for (int i = 0; i < kQPitch; ++i) column[i] = -1;
  for (int lane = 0; lane < kQCols; ++lane) {
    const int at = 2 * q_pair(lane >> 1) + (lane & 1);
    if (at < 0 || at >= kQPitch || column[at] >= 0) { std::printf("write of column %d at %d\n", lane, at); ++bad; }
    else column[at] = lane;
  }
  for (int og = 0; og < 64 / kQRows; ++og)
    for (int j = 0; j < kQPairs; ++j) {
      const int pair = q_read_pair(og, j);
      if (pair < 0 || 2 * pair + 1 >= kQPitch) { std::printf("group %d reads pair %d\n", og, pair); ++bad; continue; }
      for (int k = 0; k < 2; ++k)
        for (int o = 0; o < kQPer; ++o) {
          const int c = kQPer * og + o, tap = 2 * j + k - o;
          if (c < kQOut && tap >= 0 && tap < kQWin && column[2 * pair + k] != c + tap) {
            std::printf("output %d tap %d reads column %d\n", c, tap, column[2 * pair + k]); ++bad;
          }
        }
    }
  return bad != 0;
}
"""


def test_column_sums_stay_inside_their_row(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "tile.cpp", tmp_path / "tile"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
