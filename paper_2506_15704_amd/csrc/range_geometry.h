// Where the pieces of the range kernel's survivors lie in a head's score / position rows.
#pragma once
#include "lfps_internal.h"
#include "wide_cut.h"

namespace lfps {

// A group's rows [0, n) are cut into ranges of `range` rows and the candidates of a range into four pieces.  Piece p
// belongs to range p / 4 and keeps its survivors from start(p) on: a range's pieces stand a quarter of the range apart
// (of the last range: a quarter of its rows, rounded up to 16, which stays below n rounded up to 64).
struct RangePieces {
  int range, last, apart_last, count;
  // parts > 0: that many ranges of equal length, a multiple of 64 rows, whatever range_ is.
  __device__ __forceinline__ RangePieces(int n, int range_, int parts) : range(parts > 0 ? equal_ranges(n, parts) : range_) {
    const int ranges = n > 0 ? (int)((uint32_t)(n - 1) / (uint32_t)range) + 1 : 0;
    last = ranges - 1;
    const int rows = n - last * range;                   // of the last range
    apart_last = (((rows + 3) >> 2) + 15) & ~15;
    count = 4 * ranges;
  }
  __device__ __forceinline__ int start(int piece) const {
    const int at = piece >> 2;
    return at * range + (piece & 3) * (at == last ? apart_last : range >> 2);
  }
};

}  // namespace lfps
