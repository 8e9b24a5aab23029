"""Every byte that the wide tiles' copies read lies inside the operand, and
every row inside a ragged tile arrives at its place: the copies' address
arithmetic, compiled for the host and walked lane by lane."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2410_11720_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "wide_copy.hpp"
using namespace abft;

static long bad = 0;

// a tile of `tile` rows at row0 of an operand [rows][k] (K-major) or
// [k][rows] (MN-major), leading dimension ld elements
template <bool KM>
void operand(int rows, int k, int ld, int tile) {
  if (!wide_rows_ok(KM, rows)) { ++bad; return; }
  const unsigned ldb = unsigned(ld) * 2;
  const unsigned long end = KM ? (unsigned long)(rows - 1) * ldb + 2ul * k
                               : (unsigned long)(k - 1) * ldb + 2ul * rows;
  for (int row0 = 0; row0 < rows; row0 += tile)
    for (int k0 = 0; k0 < k; k0 += 64)
      for (int i = 0; i < tile / 8; ++i)
        for (int lane = 0; lane < 64; ++lane) {
          const unsigned long at = (unsigned long)WideRuns<KM>::lane_part(ldb, lane) +
                                   WideRuns<KM>::run_part(ldb, row0, rows, i) +
                                   (unsigned long)k0 * WideRuns<KM>::k_part(ldb);
          if (at + 16 > end) ++bad;
          // the 8 elements a lane brings, by the image's layout
          const int r = lane >> 3, c = lane & 7;
          int row, kk;
          if (KM) { row = row0 + 8 * i + r; kk = k0 + 8 * (c ^ r); }
          else { kk = k0 + 8 * (i & 7) + r; row = row0 + 64 * (i >> 3) + 8 * (c ^ (2 * (r & 3))); }
          const unsigned long want = KM ? (unsigned long)row * ldb + 2ul * kk
                                        : (unsigned long)kk * ldb + 2ul * row;
          if (row < rows && at != want) ++bad;
        }
}

void strip(int rows, int k, int ld, int row0, int runs) {
  const unsigned ldb = unsigned(ld) * 2;
  for (int i = 0; i < runs; ++i)
    for (int k0 = 0; k0 < k; k0 += 64)
      for (int lane = 0; lane < 64; ++lane) {
        const unsigned long at =
            (unsigned long)wide_strip_part(ldb, row0 + 8 * i, rows, lane) + 2ul * k0;
        if (at + 16 > (unsigned long)(rows - 1) * ldb + 2ul * k) ++bad;
        const int r = lane >> 3, row = row0 + 8 * i + r, kk = k0 + 8 * ((lane & 7) ^ r);
        if (row < rows && at != (unsigned long)row * ldb + 2ul * kk) ++bad;
      }
}

int main() {
  for (int tile : {256, 192, 128})
    for (int rows : {64, 128, 192, 256, 320, 448, 1088, 2304}) {
      operand<true>(rows, 128, 128, tile);
      operand<true>(rows, 64, 192, tile);
      operand<false>(rows, 128, rows, tile);
      operand<false>(rows, 64, rows + 64, tile);
    }
  for (int rows : {8, 32, 96, 2592}) operand<true>(rows, 64, 64, 256);
  // image rows: four per checksum block of R rows, tiles of 128 and 256
  for (int R : {32, 64, 128})
    for (int bm : {128, 256})
      for (int M : {R, 3 * R, 11 * R})
        for (int m0 = 0; m0 < M; m0 += bm)
          if (4 * bm / R <= 16) strip(4 * (M / R), 128, 192, 4 * (m0 / R), (4 * bm / R + 7) / 8);
  if (wide_rows_ok(true, 4) || wide_rows_ok(false, 96) || wide_rows_ok(true, 0)) ++bad;
  std::printf("%ld\n", bad);
  return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_copies_stay_inside_and_land_in_place(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, f"{res.stdout.strip()} reads outside or out of place"
