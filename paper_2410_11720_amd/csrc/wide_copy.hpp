// Which bytes the wide GEMM tiles copy to LDS (plain arithmetic: also
// compiled on the host, where a test walks every lane of ragged tiles).
//
// A copy's address is the descriptor's base plus a lane part plus a scalar
// part, and the hardware checks the lane part alone against the
// descriptor's size. So no row past an operand's end may be named at all:
// the runs of a ragged tile that lie past the end start at the last whole
// run instead, and what they bring is multiplied into outputs that are never
// stored.
#pragma once

#include <stdint.h>

namespace abft {

// Extents the runs fit: 8 rows of a K-major operand, 64 columns of an
// MN-major one.
constexpr bool wide_rows_ok(bool kmaj, int rows) {
  return rows > 0 && rows % (kmaj ? 8 : 64) == 0;
}

// One operand of a workgroup: rows (of M or N) by 64 of k per stage, as 1-KB
// runs. K-major images are [rows][64], 16-byte chunk c of row r at chunk
// c ^ (r & 7), a run is 8 rows; MN-major ones are 64-column sub-images
// [64 k][64], chunk c of k-row k at c ^ 2 (k & 3), a run is 8 k-rows of one.
// ldb: bytes per row in memory.
template <bool KMAJ>
struct WideRuns {
  // lane part of a run's copy: row lane / 8, the chunk that belongs at
  // chunk lane % 8
  static constexpr uint32_t lane_part(uint32_t ldb, int lane) {
    const uint32_t r = uint32_t(lane) >> 3, c = uint32_t(lane) & 7;
    return r * ldb + ((KMAJ ? c ^ r : c ^ (2 * (r & 3))) << 4);
  }
  // scalar part of run i of the tile at row0 for k = 0; `rows`: the
  // operand's extent (wide_rows_ok)
  static constexpr uint32_t run_part(uint32_t ldb, int row0, int rows, int i) {
    const int at = KMAJ ? row0 + 8 * i : row0 + 64 * (i >> 3);
    const int last = rows - (KMAJ ? 8 : 64);
    const uint32_t start = uint32_t(at < last ? at : last);
    return KMAJ ? start * ldb : uint32_t(8 * (i & 7)) * ldb + start * 2;
  }
  // bytes per step of k
  static constexpr uint32_t k_part(uint32_t ldb) { return KMAJ ? 2u : ldb; }
};

// Lane part of a strip's run of 8 image rows (K-major), the first at row0:
// rows past the image's last repeat it.
constexpr uint32_t wide_strip_part(uint32_t ldb, int row0, int rows, int lane) {
  const int r = lane >> 3, at = row0 + r, c = (lane & 7) ^ r;
  return uint32_t(at < rows ? at : rows - 1) * ldb + uint32_t(c << 4);
}

}  // namespace abft
