// How long the ranges of the range kernel are (range_score.hip): host arithmetic only, so that a test can compile it by itself.
#pragma once
#include <stdint.h>

#include "wide_cut.h"

namespace lfps {

constexpr int kRangeMax = 8192;      // rows of a range at most: a word of bitmap per thread

// Rows per range for `groups` (request, KV head) pairs of up to `rows` rows, a multiple of 64, or 0 where the separate kernels are
// faster: they cut all candidates into equal parts for two tiles in flight per wave, which wins once there is enough work to fill the
// chip.
//   From the Top-k: every workgroup reads the Top-k rows of its group, 5 us in which it loads no rows, so there may be no more rows
//   than 1024 ranges of 1024.  Steps, separate -> together: 8 groups x 32K rows 34.6 -> 28 us, 24 x 20K (paged fp16) 31.9 ->
//   23.6; but 64 x 32K 65.4 -> 69 us, paged FP8 128 x 64K 82 -> 98.  Up to the line: 0.5 to 1 million rows in 8 to 256 groups, whole
//   steps 6 to 10 us shorter (32 x 32K 55.3 -> 48.8, 256 x 4K 64.0 -> 53.8, FP8 8 x 130K, k = 4000 58.2 -> 49.3).  Ranges of 512
//   rows while that leaves at most 512 of them, else 1024 (512 to 2048 differ by 3 %).
//   From the table flags, a few words per range: candidates are 4 % of the rows, so ranges of 2048 give a wave 20 rows.
//   64 x 32K: 23.6 -> 16.1 us for the two kernels.  Up to 4 million rows.
inline int range_rows_for(int64_t groups, int rows, int heads_per_group, bool tables) {
  auto ranges = [&](int each) { return groups * ((rows + each - 1) / each); };
  int range = tables ? 2048 : (ranges(512) <= 512 ? 512 : 1024);
  if (groups * rows > (tables ? 4 << 20 : 1 << 20)) return 0;
  while ((rows + range - 1) / range > 256) range *= 2;     // at most 1024 pieces per head
  // No more than 1024 workgroups, whose fixed part (Top-k rows or flags, list, query) costs more than the rows they add: as many
  // equal ranges per group as that allows.  1024 are resident at once (four per CU) with ranges of up to 3520 rows; with four heads per
  // group LDS holds three of the longer ones, which is still the faster form.  Eight table steps with their start, ranges of 2048 ->
  // these: 64 groups x 32777 rows 594 -> 584 us, x 65509 1033 -> 1016 (one head per group 630 -> 599), 128 x 32709 1032 -> 1019, 512 x
  // 8109 1257 -> 1246; four steps from the Top-k, ranges of 1024 -> these: 200 x 5195 166 -> 139, 72 x 14505 170 -> 145, 600 x 1395
  // 191 -> 165.
  const int64_t most = 1024 / groups;
  if (most > 0 && ranges(range) > 1024 && range < kRangeMax) {
    int64_t parts = most;
    // 513 to 1023 groups get one range each, and half the chip or more its share of the rows.  With four heads per group and more than
    // 4096 rows two or three ranges are faster (from 8065 rows on four, of 2048), ranges of 2048 -> one -> these: 520 x 8009 1333 ->
    // 1341 -> 1322, 704 x 5909 1411 -> 1449 -> 1412, 560 x 7309 1322 -> 1333 -> 1311, 600 x 5009 1166 -> 1172 -> 1162; up to 4096 rows,
    // and with fewer heads, one is (800 x 3659 1245 -> 1232, two 1249; one head per group 600 x 6909 723 -> 701, three 709).
    if (parts == 1 && heads_per_group == 4 && rows > 4096) parts = (rows + 2687) / 2688;
    range = (int)(((rows + parts - 1) / parts + 63) & ~63);
  }
  return range <= kRangeMax ? range : 0;
}


// The wide form (wide_score.hip) of contexts from the Top-k that range_rows_for does not take.
struct WidePlan {
  int rows;        // of a workgroup at most in an even cut, a multiple of 64; 0: the separate kernels
  int parts;       // workgroups per group, where all requests have about as much work
  int slots;       // workgroups per KV head where they have not; 0: one request
  int most;        // of these, for one request
};

// Every workgroup reads the Top-k rows of its group once and keeps two tiles per wave in flight, so there are as many as the chip holds
// at once, 512: 1024 take 5 to 12 % longer (64 groups x 32K rows 228 -> 240 us for four steps, 128 x 128K 810 -> 853, FP8 128 x 64K 286
// -> 320), 2048 still more.  257 to 384 groups get two workgroups each, half the chip standing empty with one costs more than a second
// generation: 264 x 20000 444 -> 418, 320 x 30000 668 -> 624, 384 x 32K 783 -> 759 (480 x 20000 with two 576 -> 600).
// Four steps, separate kernels -> these: 64 groups x 32K rows 253 -> 228, 128 x 128K 884 -> 810, 16 x 66000 FP8 145 -> 108, 800 x 8000
// 514 -> 461; between 171 and 255 groups, with two workgroups each, 176 x 40000 868 -> 846, 200 x 40000 934 -> 892, 240 x 40000 1071 -> 1016.
// Up to 2^20 rows the ranges above are the better ones (1 x 32K 72 against 74, 8 x 8000 76 against 80).  More than 65536 rows a workgroup
// there cannot be (256 groups and more of longer contexts): their places have 16 bits.  Such contexts have the separate kernels.
// Requests of uneven work share the workgroups out by it.  Where they have the fewest already there are 256 more, which else return at once.
// Four steps of 8 KV heads, separate kernels (which cut the candidates of all requests into equal parts) -> the same number for every
// request -> by their work: one request of 100000 rows and 31 of 2000 317 -> 803 -> 306 us, FP8 pages 288 -> 826 -> 247, one of 131072 and
// 15 of 4096 286 -> 515 -> 265, one of 32768 and 127 of 1000 474 -> 848 -> 437, 32 x 64K with one budget of 4096 and 31 of 64 518 -> 1077 ->
// 538, 64 whose lengths fall from 32768 by a tenth each 462 -> 680 -> 500.  512 more instead of 256: 131072 and 15 x 4096 293, the
// budgets 623.
// heads: KV heads; pieces: what a head's row of piece counts holds.
inline WidePlan wide_plan_for(int batch, int heads, int rows, int pieces) {
  const int64_t groups = (int64_t)batch * heads;
  int64_t parts = groups <= 384 && groups > 256 ? 2 : 512 / groups;
  parts = parts < 1 ? 1 : (parts > 128 ? 128 : parts);                      // (two strips of four pieces, 1024 per head)
  const int64_t most = 2 * (int64_t)equal_ranges(rows, 2 * (int)parts);
  if (most > kWideMax) return WidePlan{0, 0, 0, 0};
  const int shared = batch * (int)parts, extra = batch * fewest_parts(rows) + (256 + heads - 1) / heads, of_one = pieces / 8 < 128 ? pieces / 8 : 128;
  return WidePlan{(int)most, (int)parts, batch == 1 ? 0 : (shared > extra ? shared : extra), of_one > (int)parts ? of_one : (int)parts};
}

// Its grid, see WideBlock.
struct WideGrid {
  int beside, parts, deep;
};
inline WideGrid wide_grid(const WidePlan& plan, int batch, int heads) {
  const int groups = batch * heads, beside = groups % 8 == 0 || plan.parts == 1 ? 8 : 1, row = beside * plan.parts;
  const int over = plan.slots > batch * plan.parts ? (plan.slots - batch * plan.parts) * heads : 0;
  return WideGrid{beside, plan.parts, (groups + beside - 1) / beside + (over + row - 1) / row};
}

}  // namespace lfps
