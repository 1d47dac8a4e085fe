// Which workgroup makes which part of which head's output row: arithmetic only, so that a test can compile it by itself.
#pragma once
#include "wide_cut.h"

namespace lfps {

// Workgroups per head, each for its part of the channels: one CU takes rows in at 64 bytes a cycle, and few heads leave most of the
// chip idle.  Four, while every one has a CU of its own.  Each makes the head's list, which costs no time, and the sums of a channel
// are made as by one workgroup: the same bits.  One -> four, us: steps of 1 x 32K, k = 1024 25.5 -> 24.2, exact Top-k with its
// attention 34.6 -> 33.2; steps of 1 x 128K, k = 4096 74.8 -> 66.0, 2 x 8000 FP8, k = 128 16.7 -> 16.3.  Two for 128 heads: bf16 4 x
// 32K 54.7 -> 55.0, 4 x 64K 61.9 -> 61.3, FP8 35.1 -> 34.5, not worth the kernels.  Numbers of groups that are no multiple of 8, four steps,
// one -> four on any XCD -> four on one: 12 groups x 32K, k = 1024 113.8 -> 118.9 -> 111.8, x 128K, k = 4096 384 -> 369 -> 353, FP8 97.7 ->
// 104.7 -> 95.0 and 237 -> 265 -> 227; 4 groups x 32K 80.6 -> 78.5 -> 77.0, x 128K 197.5 -> 180.6 -> 178.2, FP8 163 -> 155 -> 149.5.
// With values in host memory one: parts of a row are requests of their own over the host link (1 x 32K bf16, k = 1024, select and attention
// 152 us with one, 197 with four).
inline int attend_parts_for(int heads, bool v_on_device) { return heads <= 64 && v_on_device ? 4 : 1; }

// Workgroups are dealt to the 8 XCDs round-robin (workgroup i runs on XCD i % 8) and every XCD has its own L2.  The heads of a KV group
// select largely the same rows, so the heads * kParts workgroups of a group are given ids that differ by multiples of 8: they run on
// one XCD at about the same time and a V row (and of a row the cache line, of which a part takes a half or less) fetched for one is an L2 hit
// for the others.  Where the number of groups is no multiple of 8 some XCDs' last ids have none of them; with one workgroup a head the
// groups follow on each other then.
struct HeadPlace {
  int bg, b, g, bh;                                // KV group, request, KV head, query head (b * Hq + h)
  int in_group;                                    // which of the group's heads
  int part;                                        // which kParts-th of the output row's channels the workgroup makes
  bool none;                                       // nobody's
};
LFPS_BOTH int attend_blocks_for(int groups, int heads, int parts) { return (parts > 1 ? (groups + 7) / 8 * 8 : groups) * heads * parts; }
template <int kParts>
LFPS_BOTH HeadPlace place_of_block_for(int requests, int kv_heads, int heads, uint32_t block) {
  const int shift = heads >> 1;                    // log2 of 1, 2 or 4 heads per group
  const bool dealt = kParts > 1 || (requests * kv_heads) % 8 == 0;
  const uint32_t slot = dealt ? block >> 3 : block, head = slot / kParts;
  HeadPlace p;
  p.part = (int)(slot % kParts);
  p.in_group = (int)(head & (uint32_t)(heads - 1));
  p.bg = (int)(dealt ? (head >> shift) * 8 + (block & 7) : head >> shift);
  p.b = (int)((uint32_t)p.bg / (uint32_t)kv_heads);
  p.g = p.bg - p.b * kv_heads;
  p.bh = (p.bg << shift) + p.in_group;
  p.none = kParts > 1 && p.b >= requests;
  return p;
}

}  // namespace lfps
