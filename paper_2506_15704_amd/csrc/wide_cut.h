// Which rows of a group a workgroup of the wide kernel (wide_score.hip) has: arithmetic only, for the host and the device, so that a
// test can compile it by itself.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define LFPS_BOTH __host__ __device__ __forceinline__
#else
#define LFPS_BOTH inline
#endif

namespace lfps {

// Rows [0, n) in at most `parts` ranges of equal length, a multiple of 64.
LFPS_BOTH int equal_ranges(int n, int parts) {
  const int rows = (int)(((uint32_t)n + (uint32_t)parts - 1u) / (uint32_t)parts + 63u) & ~63;
  return rows > 64 ? rows : 64;
}

// The rows [0, n) of a group are cut into 2 * parts strips of equal length, and workgroup `part` of `parts` has the strips part and
// parts + part.  It counts its rows through: place i is row i of the first strip, place rows + i is row i of the second.
struct Strips {
  int rows;                                  // of a strip
  int first, second;                         // row where they begin
  LFPS_BOTH Strips(int n, int parts, int part) : rows(equal_ranges(n, 2 * parts)), first(part * rows), second((parts + part) * rows) {}
  LFPS_BOTH int row_of(int place) const { return place + (place < rows ? first : second - rows); }
};

// The strip [begin, begin + rows) of a request of n rows, and which windows [i - r, i + r + 1] touch it: those with touches(i).
// (i is any int32; r is at most 2^20.)
struct StripWindows {
  int begin, end, lowest;
  uint32_t span;
  LFPS_BOTH StripWindows(int n, int begin_, int rows, int r) : begin(begin_), end(n - begin_ < rows ? n : begin_ + rows) {
    const int highest = end - 1 + r < n - 1 ? end - 1 + r : n - 1;
    lowest = begin - 1 - r > 0 ? begin - 1 - r : 0;
    span = begin < n ? (uint32_t)(highest - lowest + 1) : 0u;
  }
  LFPS_BOTH bool touches(int i) const { return (uint32_t)i - (uint32_t)lowest < span; }
  // ... and the rows of the strip, counted from its first, that such a window covers
  LFPS_BOTH static int from(int i, int r, int begin) { return i - r > begin ? i - r - begin : 0; }
  LFPS_BOTH static int to(int i, int r, int begin, int end) { return (i + r + 1 < end ? i + r + 1 : end - 1) - begin; }
};

constexpr int kWideMax = 65536;      // rows of a workgroup at most: their places are 16 bits
LFPS_BOTH int fewest_parts(int n) { return n > kWideMax ? (n - 1) / kWideMax + 1 : 1; }

// Which work workgroup (x, y, z) of a grid of `beside` x `parts` x any has.  Workgroups are dealt to the XCDs in turn, and those of a
// group share an L2, so eight groups lie side by side, where they are a multiple of eight or have one workgroup each: without that
// 65535 groups and what is behind them would be more than the 65535 that a grid may be deep.
// Of an even cut it is part `part` of request b's KV head g; behind those the grid has workgroups for batches of uneven requests (`extra`).
// 256 workgroups take a CU each, and the next 256 share them: theirs are other parts, so that where the candidates crowd in one strip,
// that of all groups, two workgroups that have them don't share a CU.
struct WideBlock {
  bool extra;
  int at_extra, b, g, part;
  LFPS_BOTH WideBlock(int groups, int heads, int beside, int parts, int x, int y, int z) {
    const int at = z * beside + x;
    extra = at >= groups;
    at_extra = (z * beside - groups) * parts + (y * beside + x);
    b = extra ? 0 : (int)((uint32_t)at / (uint32_t)heads);
    g = extra ? (int)((uint32_t)at_extra % (uint32_t)heads) : at - b * heads;
    part = (int)(((uint32_t)y + ((uint32_t)(z * parts * beside) >> 8) * (uint32_t)(parts / 2)) % (uint32_t)parts);
  }
  // ... and of an uneven one the slot of that KV head, request by request.
  LFPS_BOTH int slot(int batch, int heads, int parts) const { return extra ? batch * parts + (int)((uint32_t)at_extra / (uint32_t)heads) : b * parts + part; }
};

// How many of the workgroups of a KV head a request gets.  `rows`: of its candidates, about; `all`: of those of all requests; `spare`: the
// workgroups beyond the fewest that each request can do with.  (No more than there are: what the quotients' errors add up to, below 1e-3 of
// a spare one, is less than what rounding down leaves.)  A batch is cut evenly unless a request has more than twice its share.
LFPS_BOTH bool uneven(float largest, float all, int batch) { return largest * (float)batch > 2.f * all; }
LFPS_BOTH int parts_of_request(int n, float rows, float all, int spare, int most) {
  const int parts = fewest_parts(n) + (int)((float)spare * (rows / all));
  return parts < most ? parts : most;
}

}  // namespace lfps
