// S2 — scores q . K_j / sqrt(D) of selected rows for the G query heads that share a KV head
// (Alg. 1 line 8; Sec. 1 Step 1 restricted to the candidates).  Also the dense variant over all
// rows (the exact Top-k baseline's Step 1), and a per-head variant for arbitrary index lists.
//
// The path is bound by the bytes of the K rows it gathers; the arithmetic is kept off the
// vector ALU so it cannot become the limit:
//   bf16 cache: one wave handles 16 rows at a time with v_mfma_f32_16x16x32_bf16.  The B operand
//     is the K tile exactly as it lies in memory (each lane loads 16-byte pieces of one row),
//     so a row is fetched once for all G heads.  The A operand is
//     the query: each fp32 q is split into three bf16 terms q = q0 + q1 + q2 (24 mantissa bits),
//     and A's row 4*h + t holds term t of head h.  bf16 x bf16 products are exact in fp32, so
//     the sum D[4h+0] + D[4h+1] + D[4h+2] is the fp32-accumulated dot product with the fp32
//     query; it lands in lane group h without any cross-lane reduction.
//   fp16 cache: the same with v_mfma_f32_16x16x32_f16; the query terms are fp16 too, the second and third
//     scaled up by 2^11 and 2^22 so that they stay normal numbers, and scaled back when the three
//     D rows are added (fp16 x fp16 products are exact in fp32 as well).  |q| must stay below 65504.
//   fp32 cache: 16 lanes per row, 8 channels each, fp32 FMAs and a reduce by lane permutations.
#include "candidates.h"
#include "score_mfma.h"

namespace lfps {

// ----------------------------------------------------------------------------- bf16 / fp16 / fp8, MFMA
// grid: (tiles_x, B*Hkv).  GATHER: rows come from cand[bg, 0:count]; else rows are 0..n_b-1.
//
// Lane (j, kb) = (lane & 15, lane >> 4) supplies column j of the B operand: for MFMA step kk it
// loads the 16-byte chunk kk + 4*kb of row j, i.e. every lane walks its own contiguous 64 bytes of
// the row over the four steps (measured faster than splitting a row into four 64-byte quarters
// per step: all four loads of a tile touch both cache lines of every row).  Any assignment of
// channels to (kk, kb) is valid as long as the A operand uses the same one.
// The row ids of the next iteration are fetched, and the scores of the previous iteration stored,
// right after this iteration's loads are issued.
template <int G, bool GATHER, bool kPaged, int kKind>
__global__ __launch_bounds__(kScoreThreads) void k_group_score_bf16(Shape s, const float* __restrict__ q,
                                                                    const void* __restrict__ K, int64_t stride_b,
                                                                    int64_t stride_h, int64_t stride_n, KvPage pg,
                                                                    const int32_t* __restrict__ seq_lens,
                                                                    const int32_t* __restrict__ cand,
                                                                    const int32_t* __restrict__ cand_count,
                                                                    float* __restrict__ score, int64_t score_stride,
                                                                    float scale, int32_t* __restrict__ flags,
                                                                    float* __restrict__ tops,
                                                                    const int32_t* __restrict__ kk) {
  request_arguments<decltype(&k_group_score_bf16<G, GATHER, kPaged, kKind>)>();
  const int bg = blockIdx.y, b = bg / s.Hkv, g = bg % s.Hkv;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = lane & 15, kb = lane >> 4;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  int count = GATHER ? cand_count[bg] : n;
  if (GATHER) count = count < 0 ? 0 : (count > s.cand_cap ? s.cand_cap : count);
  const int first = (blockIdx.x * 4 + wave) * kRowsPerWaveIter;
  if (first >= count) return;

  using Op = typename KTile<kKind>::Operand;
  Op A[4];
  report_q_range(load_query_operand(A, q, (int64_t)b * s.Hq + (int64_t)g * G, G, j, kb), flags);

  using Rows = RowMap<kPaged>;
  constexpr int ES = KTile<kKind>::kElemBytes;
  const char* Kbg = static_cast<const char*>(K) + Rows::base(b, g, stride_b, stride_h) * ES;
  const int32_t* cbg = GATHER ? cand + (int64_t)bg * s.cand_cap : nullptr;
  float* sc = score + ((int64_t)b * s.Hq + (int64_t)g * G + kb) * score_stride;   // lane group kb -> head kb
  float* my_tops = nullptr;
  if constexpr (!GATHER) {
    if (tops && select_takes_tops(s, n, kk[b])) my_tops = tops + ((int64_t)b * s.Hq + (int64_t)g * G + kb) * (score_stride >> 4);
  }
  score_slots_mfma<kPaged, kKind, !GATHER>(A, Kbg, pg, b, stride_b, stride_n, [&](int slot) { return GATHER ? cbg[slot] : slot; }, n, count, first,
                                           (int)gridDim.x * 4 * kRowsPerWaveIter, sc, kb < G, scale, my_tops);
}

// ----------------------------------------------------------------------------- bf16 / fp16 / fp8, MFMA, filtered output
// The same scoring, but only rows whose score reaches a per-head threshold are written out
// (the threshold is the previous step's k-th best score minus a margin: consecutive decode steps
// select almost the same rows, the premise of the method).  Writing every score costs far more
// than its share of bytes because the small writes interleave with the row gather; survivors are
// a few per cent of the rows.
//
// Work split: the candidate slots of all groups, laid end to end, form one line [0, total); it is
// cut into equal parts of S slots, one per wave of the launch, and the launch has exactly as many
// waves as the chip holds at once.  Every wave therefore reads the same number of rows whatever
// the mix of sequence lengths, and no workgroup waits for a slot.  The candidates kernel has given
// every group its place on the line (group_start; the order of the groups on the line is the
// order in which they finished there, which changes nothing in the result) and left the line's
// length in *line_total.  A part that crosses a group boundary is handled as several pieces, one
// per group.  Piece `seg` of a group (seg = wave index minus the index of the first wave that
// touches the group) covers the group's slots [lo, hi) and appends its survivors (score, row
// position), in slot order, at offset lo of each head's score / position rows (staged in LDS,
// written when the piece is done); their number goes to seg_count[head, seg].  No atomics here:
// the lists are ascending in position and the same from run to run.
// A threshold of -inf keeps every row; NaN means there is no previous step.
//
// How the rows are fetched.  Bound by the bytes of the rows.  Candidates of more than kKeptBytes cannot be found again in the
// memory-side cache (256 MB) by the next step, so their rows are read past the caches (StreamTile): 128 groups x 128K rows,
// 954 MB of candidates 193 -> 175 us; all rows of 64 groups x 64K (kDense), 1.07 GB 185 -> 162.5 us = 6.6 TB/s; and what the select
// reads after it (the survivors, V rows shared by the heads of a group) is no longer driven out: its kernel 40 -> 31 us.
// (Non-temporal loads of KTile's shape fetch every line several times, 300 us; StreamTile with ordinary loads gains nothing, 196
// us.)  Up to kKeptBytes ordinary loads, every lane its own channels (KTile): where the same layer's steps follow each other, the
// next one finds nine tenths of its rows in the cache.  64 groups x 32K rows, 220 MB: a step 64 us, 66 past the caches.  Two steps
// of 16 requests, kept -> past: 260 MB of bf16 candidates 152.3 -> 152.0 us, 275 MB 161.0 -> 157.7; FP8 260 MB 168.0 -> 169.7,
// 275 MB 176.0 -> 174.8.
// The parts are cut at multiples of 16 slots: of 64, a part of 420 slots grew by 6 % and the last waves had nothing to do
// (64 groups x 32K rows: 38.1 -> 37.0 us).
constexpr int kFilterStage = 256;   // survivors one wave can hold per head before it must write them out

// kDense: the "candidates" of a group are all its rows 0..count-1 (no list is read): the exact Top-k baseline's
// scoring pass with a threshold from a sample of the rows.
template <int G, bool kPaged, int kKind, bool kDense>
__global__ __launch_bounds__(kScoreThreads, 2) void k_filter_score_bf16(
    Shape s, const float* __restrict__ q, const void* __restrict__ K, int64_t stride_b, int64_t stride_h,
    int64_t stride_n, KvPage page, const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ cand,
    const int32_t* __restrict__ cand_count, const int64_t* __restrict__ group_start,
    const int64_t* __restrict__ line_total, const float* __restrict__ thr_state, float margin, float* __restrict__ tau_out,
    const int32_t* __restrict__ skip_if, float* __restrict__ score, int32_t* __restrict__ slot_out, int64_t score_stride,
    int32_t* __restrict__ seg_count, int32_t* __restrict__ seg_rows_out, int min_seg_rows, int nseg, float scale,
    int32_t* __restrict__ flags) {
  __shared__ float stage_score[4][G][kFilterStage];
  __shared__ int32_t stage_slot[4][G][kFilterStage];
  __shared__ u32x4 turn[4][StreamTile<kKind>::kLdsChunks];
  request_arguments<decltype(&k_filter_score_bf16<G, kPaged, kKind, kDense>)>();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform values stay in scalar registers
  const int j = lane & 15, kb = lane >> 4;
  const int n_groups = s.B * s.Hkv;

  // Before the first row there is a chain of loads, each written by another kernel and a trip to memory of about 0.8 us: the
  // line and the groups' places on it together, then row ids, threshold and length together, (the block table,) the rows.
  // (Waits that the compiler would put in between are avoided by asking for everything of a link before any of it is used.)
  struct Places {
    int64_t st[4];
    int cnt[4];
  };
  auto places_from = [&](int g0) {
    Places p;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int at = g0 + 64 * u + lane;
      p.st[u] = at < n_groups ? group_start[at] : 0;
      p.cnt[u] = at < n_groups ? cand_count[at] : 0;
    }
    return p;
  };
  Places at_hand = places_from(0);
  // ---- the part of this wave: S slots from wave_index * S; every wave derives the same S
  const int64_t total = *line_total;
#pragma unroll
  for (int u = 0; u < 4; ++u) asm volatile("" : "+v"(at_hand.cnt[u]));
  const int n_waves = (int)gridDim.x * 4;
  int64_t S = (total >> 30) == 0 ? (int64_t)(((uint32_t)total + (uint32_t)n_waves - 1u) / (uint32_t)n_waves)
                                 : (total + n_waves - 1) / n_waves;
  S = (S + 15) & ~(int64_t)15;
  S = S < min_seg_rows ? min_seg_rows : S;
  if (blockIdx.x == 0 && tid == 0) *seg_rows_out = (int32_t)S;      // the select reads it
  const int64_t w = (int64_t)blockIdx.x * 4 + wave;
  const int64_t part_lo = w * S;
  const int64_t part_hi = part_lo + S < total ? part_lo + S : total;
  if (part_lo >= total) return;                          // nothing left for this wave
  const bool stream = total * (kD * KTile<kKind>::kElemBytes) > (kDense ? kKeptStreamBytes : kKeptBytes);

  const uint32_t below = (1u << j) - 1u;                // lanes of my 16-lane group with a lower row
  float* st_s = stage_score[wave][kb < G ? kb : 0];
  int32_t* st_i = stage_slot[wave][kb < G ? kb : 0];
  constexpr int T = kRowsPerWaveIter;

  // the groups that overlap my part: 256 groups are tested at a time, four per lane, all loads issued together; the place and
  // count of the first one found stay, those of a further one are read again (scalar loads that hit the cache)
  auto count_of = [&](int c) { return c < 0 ? 0 : (c > s.cand_cap ? s.cand_cap : c); };
  for (int g0 = 0;;) {
    uint64_t hits[4];
    int found = -1, found_count = 0;
    int64_t found_start = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t st = at_hand.st[u];
      const int cnt = count_of(at_hand.cnt[u]);
      hits[u] = __ballot(cnt > 0 && st < part_hi && st + cnt > part_lo);
      if (found < 0 && hits[u]) {
        const int src = __builtin_ctzll(hits[u]);
        found = g0 + 64 * u + src;
        found_count = __builtin_amdgcn_readlane(cnt, src);
        found_start = ((int64_t)__builtin_amdgcn_readlane((int)(st >> 32), src) << 32) |
                      (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)st, src);
      }
    }
  while (hits[0] | hits[1] | hits[2] | hits[3]) {         // one piece per overlapping group
    int bg = 0;
#pragma unroll
    for (int u = 3; u >= 0; --u) bg = hits[u] ? g0 + 64 * u + __builtin_ctzll(hits[u]) : bg;
#pragma unroll
    for (int u = 3; u >= 0; --u) {
      bool earlier = false;
#pragma unroll
      for (int v = 0; v < u; ++v) earlier |= hits[v] != 0;
      if (!earlier) hits[u] &= hits[u] - 1;
    }
    const int64_t pg = bg == found ? found_start : group_start[bg];      // the group's place on the line
    const int count = bg == found ? found_count : count_of(cand_count[bg]);
    const int seg_lo = part_lo > pg ? (int)(part_lo - pg) : 0;
    const int seg_hi = part_hi - pg < count ? (int)(part_hi - pg) : count;
    const int seg = (int)w - ((pg >> 31) == 0 ? (int)((uint32_t)pg / (uint32_t)S) : (int)(pg / S));

    const int b = bg / s.Hkv, g = bg % s.Hkv;
    // Slots past the end of the piece read the id of its last slot (a valid row) and are never kept:
    // no load of the loop below sits behind a branch, so the waits the compiler derives for the
    // two tiles in flight are exact counts instead of "everything outstanding".
    const int32_t* cbg = cand + (int64_t)bg * s.cand_cap;
    auto fetch_ids = [&](int base_slot) {
      const int sl = base_slot + lane;
      const int at = sl < seg_hi ? sl : seg_hi - 1;
      if constexpr (kDense) return at;
      else return cbg[at];
    };
    int ids_first = fetch_ids(seg_lo), ids_second = fetch_ids(seg_lo + T), ids_third = fetch_ids(seg_lo + 2 * T);
    int n = seq_lens[b];
    n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
    const int64_t head = (int64_t)b * s.Hq + (int64_t)g * G + (kb < G ? kb : 0);
    // NaN in thr_state = "no previous step": skip the group here, the unfiltered pass will take it.  (A bypassed head keeps
    // nothing, and needs no step before this one.)
    const float thr = thr_state[head];
    const bool skipped = skip_if && skip_if[head] != 0;
    // FP8: the query is asked for with the ids.  Loads complete in order, and asked for behind the first tile it keeps the second
    // one waiting for that (four steps of 128 groups x 64K rows 327 -> 324 us); two 16-bit tiles leave no registers for it.
    using Op = typename KTile<kKind>::Operand;
    constexpr bool kQueryFirst = kKind == kKindFp8;
    const int64_t head0 = (int64_t)b * s.Hq + (int64_t)g * G;
    QueryRows query;
    if constexpr (kQueryFirst) query.load(q, head0, G, j, kb);
    asm volatile("" : "+v"(ids_first), "+v"(ids_second), "+v"(ids_third));
    if (__ballot(kb < G && !skipped && isnan(thr))) {
      if (j == 0 && kb < G) seg_count[head * nseg + seg] = 0;
      continue;
    }
    const float tau = kb < G && !skipped ? thr - margin : INFINITY;

    using Rows = RowMap<kPaged>;
    Op A[4];
    auto take_query = [&]() {                           // (behind the first tile: overlaps its latency)
      if constexpr (!kQueryFirst) query.load(q, head0, G, j, kb);
      report_q_range(query.operand(A, G, j), flags);
    };
    constexpr int ES = KTile<kKind>::kElemBytes;
    const char* Kbg = static_cast<const char*>(K) + Rows::base(b, g, stride_b, stride_h) * ES;
    int run = 0;                                        // survivors of my head already in global memory
    int staged = 0;                                     // survivors of my head waiting in LDS

    // Survivors are staged in LDS and written out when the piece is done (or the stage is nearly
    // full).  Global stores inside the loop would share the vector-memory counter with the row
    // loads, so that every wait for a load would also wait for the stores before it.
    auto flush = [&]() {
      wave_lds_order();
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const int cnt_h = __shfl(staged, 16 * h);
        const int run_h = __shfl(run, 16 * h);
        float* dsc = score + ((int64_t)b * s.Hq + (int64_t)g * G + h) * score_stride + seg_lo + run_h;
        int32_t* dsl = slot_out + ((int64_t)b * s.Hq + (int64_t)g * G + h) * score_stride + seg_lo + run_h;
        for (int e = lane; e < cnt_h; e += 64) {
          dsc[e] = stage_score[wave][h][e];
          dsl[e] = stage_slot[wave][h][e];
        }
      }
      run += staged;
      staged = 0;
      wave_lds_order();
    };

    // Two 64-row tiles are kept in flight per wave: while tile i is multiplied, the loads of tile
    // i+1 (issued before) are still arriving.
    // phys: the tile's 64 rows as physical rows, one per lane
    auto issue = [&](auto& Bt, int phys) {
      Bt.fetch(Kbg, phys, lane, [&](int p) { return Rows::offset(page, p, stride_b, stride_n) * ES; });
    };
    auto lookup = [&](int ids) { return Rows::phys(page, b, ids); };
    // ids: their row positions
    auto consume = [&](const auto& Bt, int ids, int base_slot) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const KSub<kKind> sub = Bt.sub(t, turn[wave], lane);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          acc = mfma16(A[kk], sub.operand(kk), acc);
        const float v = Split3<Op>::sum(acc) * scale;
        const int slot = base_slot + 16 * t + j;
        const bool pass = kb < G && slot < seg_hi && v >= tau;
        const uint32_t gm = (uint32_t)(__ballot(pass) >> (16 * kb)) & 0xFFFFu;   // my head's 16 rows
        const int row = lane_value(ids, j, 16 * t);
        if (pass) {
          const int o = staged + __popc(gm & below);
          st_s[o] = v;
          st_i[o] = row;                                // the row position itself: the select needs no lookup
        }
        staged += __popc(gm);
      }
      // room for one more tile (64 rows) in every head's stage?  (wave-uniform test)
      if (__ballot(staged > kFilterStage - kRowsPerWaveIter)) flush();
    };
    auto checked = [&](int ids) { return ids < 0 || ids >= n ? 0 : ids; };   // (a bad entry of a caller's list reads row 0)

    // Row ids are fetched three tiles ahead, always BEFORE the loads of the tile that precedes
    // their use are issued: a wait for ids then never has to wait for a tile still in flight
    // (the vector-memory counter completes in issue order).
    auto walk = [&](auto Bt0, auto Bt1) {               // (the two tiles in flight)
    int base_slot = seg_lo;
    if constexpr (!kPaged) {
      int ids_0 = checked(ids_first), ids_1;              // ids of the even tile in flight, of the odd one
      int ids_b = ids_second;                             // ids of the next odd tile
      int ids_a = ids_third;                              // ids of the next even tile
      issue(Bt0, ids_0);
      take_query();
      for (; base_slot + 2 * T < seg_hi; base_slot += 2 * T) {   // at least three tiles left: no conditions inside
        issue(Bt1, ids_1 = checked(ids_b));
        ids_b = fetch_ids(base_slot + 3 * T);
        consume(Bt0, ids_0, base_slot);
        issue(Bt0, ids_0 = checked(ids_a));
        ids_a = fetch_ids(base_slot + 4 * T);
        consume(Bt1, ids_1, base_slot + T);
      }
      if (base_slot + T < seg_hi) {                       // two tiles left (wave-uniform)
        issue(Bt1, ids_1 = checked(ids_b));
        consume(Bt0, ids_0, base_slot);
        consume(Bt1, ids_1, base_slot + T);
      } else {
        consume(Bt0, ids_0, base_slot);
      }
    } else {
      // Paged cache: a block-table lookup sits between a row id and its address.  A wait completes
      // everything older than what it waits for, so with tile i in flight every step issues, BEFORE
      // the loads of tile i+1: the ids of tile i+3 and the lookup for tile i+2 (whose ids were fetched
      // one step earlier, before the loads of tile i).
      int ids_0 = checked(ids_first), ids_1 = checked(ids_second);
      int phys_0 = lookup(ids_0), phys_1 = lookup(ids_1);
      int in_0 = ids_0, in_1;                             // of the tiles in flight
      {
        const int at = phys_0;
        ids_0 = ids_third;
        issue(Bt0, at);
      }
      take_query();
      // here and at the top of every iteration: (ids_1, phys_1) describe the next odd tile, ids_0 the next even one
      for (; base_slot + 2 * T < seg_hi; base_slot += 2 * T) {
        {
          const int at = phys_1;
          in_1 = ids_1;
          ids_1 = fetch_ids(base_slot + 3 * T);
          ids_0 = checked(ids_0);
          phys_0 = lookup(ids_0);
          __builtin_amdgcn_sched_barrier(0);    // the instruction scheduler must not move these two loads
          issue(Bt1, at);                       // behind the tile's: the order is what the waits rely on
        }
        consume(Bt0, in_0, base_slot);
        {
          const int at = phys_0;
          in_0 = ids_0;
          ids_0 = fetch_ids(base_slot + 4 * T);
          ids_1 = checked(ids_1);
          phys_1 = lookup(ids_1);
          __builtin_amdgcn_sched_barrier(0);
          issue(Bt0, at);
        }
        consume(Bt1, in_1, base_slot + T);
      }
      if (base_slot + T < seg_hi) {
        issue(Bt1, phys_1);
        consume(Bt0, in_0, base_slot);
        consume(Bt1, ids_1, base_slot + T);
      } else {
        consume(Bt0, in_0, base_slot);
      }
      // A use of the prefetched ids on every path: without it the compiler moves the prologue's fetch of
      // ids_0 down to the loop entry, behind the first tile's loads, and the loop's first wait for it
      // becomes a wait for everything.
      asm volatile("" ::"v"(ids_0), "v"(ids_1));
    }
    };
    if (stream) walk(StreamTile<kKind>{}, StreamTile<kKind>{});
    else walk(KTile<kKind>{}, KTile<kKind>{});
    flush();
    if (j == 0 && kb < G) {
      seg_count[head * nseg + seg] = run;
      if (seg == 0) tau_out[head] = thr - margin;
    }
  }
    g0 += 256;
    if (g0 >= n_groups) break;
    at_hand = places_from(g0);
  }
}

// ----------------------------------------------------------------------------- fp32, vector ALU
// A wave takes 16 rows at a time, 16 lanes per row, all of its loads issued together and the ids of its next 16 rows behind
// them; the dot products are summed over the lanes without LDS.  With 64 rows per wave in four batches one wave after
// the other waited for memory four times, and few candidates made few waves: 11.2 us for 770 candidates of 8 groups, this
// way 3.6 us (a step of 1 x 4096: 24.1 -> 18.4).
constexpr int kRowsPerWaveF32 = 16;

// Scores of the slots first .. first + 15, first + step ..., below count, by one wave.  row_at(slot): the row of a slot (called
// by the lanes 0 .. 15 of a visit); an entry outside [0, n) reads row 0 and scores -inf: it ranks below every row.  sc: the score
// row of the group's first head.
template <int G, bool kPaged, typename RowAt>
__device__ __forceinline__ void score_slots_f32(const float (&qr)[G][8], const float* Kbg, const KvPage& pg, int b, int64_t stride_b,
                                                int64_t stride_n, int n, int count, int first, int step, float* __restrict__ sc,
                                                int64_t score_stride, float scale, RowAt row_at) {
  const int lane = threadIdx.x & 63;
  const int j = lane & 15, rs = lane >> 4;     // 16 lanes per row, 4 rows per wave instruction
  using Rows = RowMap<kPaged>;
  auto fetch = [&](int base) { return lane < kRowsPerWaveF32 && base + lane < count ? row_at(base + lane) : -1; };
  auto physical = [&](int row) { return Rows::phys(pg, b, row >= 0 && row < n ? row : 0); };
  int my_row = fetch(first);
  int my_phys = physical(my_row);
  for (int base = first; base < count; base += step) {
    bool ok[4];
    float4 x0[4], x1[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int row = __shfl(my_row, 4 * t + rs);
      ok[t] = row >= 0 && row < n;
      const float4* p = reinterpret_cast<const float4*>(Kbg + Rows::offset(pg, __shfl(my_phys, 4 * t + rs), stride_b, stride_n)) + 2 * j;
      x0[t] = p[0];
      x1[t] = p[1];
    }
    my_row = fetch(base + step);
    my_phys = physical(my_row);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float v = 0.f;
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float a = qr[h][0] * x0[t].x;
        a = fmaf(qr[h][1], x0[t].y, a);
        a = fmaf(qr[h][2], x0[t].z, a);
        a = fmaf(qr[h][3], x0[t].w, a);
        a = fmaf(qr[h][4], x1[t].x, a);
        a = fmaf(qr[h][5], x1[t].y, a);
        a = fmaf(qr[h][6], x1[t].z, a);
        a = fmaf(qr[h][7], x1[t].w, a);
        a = row16_butterfly_sum(a);
        v = j == h ? a : v;
      }
      const int slot = base + 4 * t + rs;
      if (slot < count && j < G) sc[(int64_t)j * score_stride + slot] = ok[t] ? v * scale : -INFINITY;
    }
  }
}

template <int G, bool GATHER, bool kPaged>
__global__ __launch_bounds__(kScoreThreads) void k_group_score_f32(Shape s, const float* __restrict__ q,
                                                                   const float* __restrict__ K, int64_t stride_b,
                                                                   int64_t stride_h, int64_t stride_n, KvPage pg,
                                                                   const int32_t* __restrict__ seq_lens,
                                                                   const int32_t* __restrict__ cand,
                                                                   const int32_t* __restrict__ cand_count,
                                                                   float* __restrict__ score, int64_t score_stride,
                                                                   float scale, int32_t* __restrict__ flags, float*, const int32_t*) {
  const int bg = blockIdx.y, b = bg / s.Hkv, g = bg % s.Hkv;
  const int wave = threadIdx.x >> 6, j = threadIdx.x & 15;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  int count = GATHER ? cand_count[bg] : n;
  if (GATHER) count = count < 0 ? 0 : (count > s.cand_cap ? s.cand_cap : count);
  const int first = (blockIdx.x * 4 + wave) * kRowsPerWaveF32;
  if (first >= count) return;

  const int64_t head0 = (int64_t)b * s.Hq + (int64_t)g * G;
  float qr[G][8];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float* qh = q + (head0 + h) * kD + 8 * j;
#pragma unroll
    for (int c = 0; c < 8; ++c) qr[h][c] = qh[c];
  }
  const float* Kbg = K + RowMap<kPaged>::base(b, g, stride_b, stride_h);
  const int32_t* cbg = GATHER ? cand + (int64_t)bg * s.cand_cap : nullptr;
  score_slots_f32<G, kPaged>(qr, Kbg, pg, b, stride_b, stride_n, n, count, first, gridDim.x * 4 * kRowsPerWaveF32,
                             score + head0 * score_stride, score_stride, scale, [&](int slot) { return GATHER ? cbg[slot] : slot; });
}

// S1 and S2 of a step over fp32 rows in one kernel: each of the gridDim.x workgroups of a group builds the group's bitmap of
// candidates, counts them, and lists and scores its part of them, slots [part * per, (part + 1) * per) of the ascending list.  List,
// count and scores are those of k_candidates and k_group_score_f32, to the bit.  Bound by latency: as two
// kernels a step of 8 groups x 4096 rows took 18.3 us in all, this way 17.0.
template <int G, bool kPaged>
__global__ __launch_bounds__(kScoreThreads) void k_candidates_score_f32(
    Shape s, const float* __restrict__ q, const float* __restrict__ K, int64_t stride_b, int64_t stride_h, int64_t stride_n,
    KvPage pg, const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ prev_topk, const int32_t* __restrict__ kk,
    int32_t* __restrict__ cand, int32_t* __restrict__ cand_count, float* __restrict__ score, int64_t score_stride, float scale,
    int32_t* __restrict__ flags) {
  request_arguments<decltype(&k_candidates_score_f32<G, kPaged>)>();
  extern __shared__ uint32_t lds[];                      // the bitmap, then the part's list
  __shared__ int wave_tot[4];
  const int bg = blockIdx.y, b = bg / s.Hkv, g = bg % s.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 15;
  const int64_t head0 = (int64_t)b * s.Hq + (int64_t)g * G;
  int n = seq_lens[b];
  int kb = kk[b];
  float qr[G][8];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float* qh = q + (head0 + h) * kD + 8 * j;
#pragma unroll
    for (int c = 0; c < 8; ++c) qr[h][c] = qh[c];
  }
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  kb = kb < 0 ? 0 : (kb > s.kmax ? s.kmax : kb);
  const int words = (s.Lcap + 31) >> 5;
  bitmap_from_topk<kScoreThreads>(s, lds, words, prev_topk + head0 * s.kmax, n, kb);
  uint32_t bits = tid < words ? lds[tid] : 0u;           // a word per thread, see kFusedRowsF32
  const int mine = __popc(bits);
  const int inc = wave_inclusive_sum(mine);
  if (lane == 63) wave_tot[wave] = inc;
  __syncthreads();
  int at = inc - mine, total = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const int t = wave_tot[w];
    at += w < wave ? t : 0;
    total += t;
  }
  const int count = total < s.cand_cap ? total : s.cand_cap;
  if (blockIdx.x == 0 && tid == 0) {
    if (total > s.cand_cap) atomicOr(flags, LFPS_FLAG_CAND_OVERFLOW);
    cand_count[bg] = count;
  }
  const int per = ((count + (int)gridDim.x - 1) / (int)gridDim.x + kRowsPerWaveF32 - 1) & ~(kRowsPerWaveF32 - 1);
  const int s0 = (int)blockIdx.x * per, s1 = s0 + per < count ? s0 + per : count;
  if (s0 >= s1) return;                                  // (workgroup-uniform)
  int32_t* list = reinterpret_cast<int32_t*>(lds + words);
  int32_t* out = cand + (int64_t)bg * s.cand_cap;
  if (at + mine <= s0) bits = 0u;
  for (; bits && at < s1; bits &= bits - 1, ++at) {
    if (at < s0) continue;
    const int row = (tid << 5) + __ffs(bits) - 1;
    list[at - s0] = row;
    out[at] = row;
  }
  __syncthreads();
  const int first = s0 + wave * kRowsPerWaveF32;
  if (first >= s1) return;
  score_slots_f32<G, kPaged>(qr, K + RowMap<kPaged>::base(b, g, stride_b, stride_h), pg, b, stride_b, stride_n, n, s1, first,
                             4 * kRowsPerWaveF32, score + head0 * score_stride, score_stride, scale,
                             [&](int slot) { return list[slot - s0]; });
}

// ----------------------------------------------------------------------------- per-head index lists
// Scores of idx[b,h,0:k_b] against q[b,h]; 16 lanes per row.  Used only when the caller of the
// sparse attention does not supply scores.  grid: (ceil(kmax/256), B*Hq).
template <typename T, bool kPaged>
__global__ __launch_bounds__(256) void k_head_score(Shape s, const float* __restrict__ q, const T* __restrict__ K,
                                                    int64_t stride_b, int64_t stride_h, int64_t stride_n, KvPage pg,
                                                    const int32_t* __restrict__ seq_lens,
                                                    const int32_t* __restrict__ idx, const int32_t* __restrict__ kk,
                                                    float* __restrict__ out, float scale) {
  const int bh = blockIdx.y, b = bh / s.Hq, h = bh % s.Hq, g = h / s.G;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = lane & 15, rs = lane >> 4;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  int kb = kk[b];
  kb = kb < 0 ? 0 : (kb > s.kmax ? s.kmax : kb);
  const int base = (blockIdx.x * 4 + wave) * 64;
  if (base >= kb) return;
  float qr[8];
  const float* qh = q + (int64_t)bh * kD + 8 * j;
#pragma unroll
  for (int c = 0; c < 8; ++c) qr[c] = qh[c];
  using Rows = RowMap<kPaged>;
  const T* Kbg = K + Rows::base(b, g, stride_b, stride_h);
  const int my_row = (base + lane < kb) ? idx[(int64_t)bh * s.kmax + base + lane] : -1;
  const bool my_ok = my_row >= 0 && my_row < n;
  const int my_phys = Rows::phys(pg, b, my_ok ? my_row : 0);
  for (int t = 0; t < 16; ++t) {
    const bool ok = __shfl((int)my_ok, 4 * t + rs) != 0;
    const int prow = __shfl(my_phys, 4 * t + rs);
    const T* p = Kbg + Rows::offset(pg, prow, stride_b, stride_n) + 8 * j;
    float x[8];
    load8(p, x);
    float a = qr[0] * x[0];
#pragma unroll
    for (int c = 1; c < 8; ++c) a = fmaf(qr[c], x[c], a);
    a = row16_butterfly_sum(a);
    int slot = base + 4 * t + rs;
    if (j == 0 && slot < kb) out[(int64_t)bh * s.kmax + slot] = ok ? a * scale : -INFINITY;
  }
}

// ----------------------------------------------------------------------------- launchers
template <int G, bool GATHER>
static hipError_t launch_gs(const Shape& s, int dtype, const float* q, const KvView& kv, const int32_t* cand,
                            const int32_t* cand_count, float* score, int64_t score_stride, int32_t* flags,
                            hipStream_t st, float* tops, const int32_t* k) {
  const int rows_max = GATHER ? s.cand_cap : s.Lcap;
  const int per_block = 4 * (dtype == LFPS_F32 ? kRowsPerWaveF32 : kRowsPerWaveIter);
  int tiles = (rows_max + per_block - 1) / per_block;
  // about four workgroups (16 waves; fp32: six, with smaller tiles) per CU, all resident at once, but no more than there
  // are tiles
  int want = (256 * (dtype == LFPS_F32 ? 6 : 4) + s.B * s.Hkv - 1) / (s.B * s.Hkv);
  int gx = tiles < want ? tiles : want;
  if (gx < 1) gx = 1;
  dim3 grid(gx, s.B * s.Hkv), block(kScoreThreads);
  const float scale = 0.08838834764831845f;   // 1/sqrt(128)
#define LFPS_LAUNCH_GS(KERNEL, TYPE, ...)                                                                          \
  hipLaunchKernelGGL((KERNEL<G, GATHER, __VA_ARGS__>), grid, block, 0, st, s, q, (const TYPE*)kv.k, kv.stride_b,   \
                     kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, cand, cand_count, score, score_stride, scale, \
                     flags, tops, k)
  const bool paged = kv.page.table != nullptr;
  if (dtype == LFPS_BF16 && kv.k_fp8) {
    if (paged) LFPS_LAUNCH_GS(k_group_score_bf16, void, true, kKindFp8);
    else LFPS_LAUNCH_GS(k_group_score_bf16, void, false, kKindFp8);
  } else if (dtype == LFPS_BF16) {
    if (paged) LFPS_LAUNCH_GS(k_group_score_bf16, void, true, kKindBf16);
    else LFPS_LAUNCH_GS(k_group_score_bf16, void, false, kKindBf16);
  } else if (dtype == LFPS_F16) {
    if (paged) LFPS_LAUNCH_GS(k_group_score_bf16, void, true, kKindF16);
    else LFPS_LAUNCH_GS(k_group_score_bf16, void, false, kKindF16);
  } else {
    if (paged) LFPS_LAUNCH_GS(k_group_score_f32, float, true);
    else LFPS_LAUNCH_GS(k_group_score_f32, float, false);
  }
#undef LFPS_LAUNCH_GS
  return hipGetLastError();
}

hipError_t launch_group_score(const Shape& s, int dtype, const float* q, const KvView& kv, const int32_t* cand,
                              const int32_t* cand_count, float* score, int64_t score_stride, int32_t* flags,
                              hipStream_t st, float* tops, const int32_t* k) {
  const bool gather = cand != nullptr;
  switch (s.G) {
    case 1: return gather ? launch_gs<1, true>(s, dtype, q, kv, cand, cand_count, score, score_stride, flags, st, tops, k)
                          : launch_gs<1, false>(s, dtype, q, kv, cand, cand_count, score, score_stride, flags, st, tops, k);
    case 2: return gather ? launch_gs<2, true>(s, dtype, q, kv, cand, cand_count, score, score_stride, flags, st, tops, k)
                          : launch_gs<2, false>(s, dtype, q, kv, cand, cand_count, score, score_stride, flags, st, tops, k);
    case 4: return gather ? launch_gs<4, true>(s, dtype, q, kv, cand, cand_count, score, score_stride, flags, st, tops, k)
                          : launch_gs<4, false>(s, dtype, q, kv, cand, cand_count, score, score_stride, flags, st, tops, k);
    default: return hipErrorInvalidValue;
  }
}

// Workgroups of k_candidates_score_f32 that share a group, or 0 where the separate kernels are faster: every
// workgroup reads the Top-k rows of its group and builds the whole bitmap, which the rows of a long context do not pay for.  The line
// is a word of bitmap per thread (beyond, half the threads count and list two words each and the others none).  Two
// workgroups per CU: more of them repeat the bitmap, fewer wait longer for their rows.  Two steps, separate -> together, us: 8 groups x
// 2000 rows 34.8 -> 31.6, x 4096 36.5 -> 34.0, x 8180 45.5 -> 40.0 (k = 2250 98.2 -> 97.0), x 9000 43.1 -> 43.7 (105.1 -> 107.3), x
// 32K 74.4 -> 80.8; 128 x 4000 63.5 -> 57.5, 128 x 8000 96.7 -> 90.5, 256 x 4000 103.5 -> 98.7; with 1024 workgroups 8 x 8000 40.6,
// with 256 256 x 4000 102.7.
static constexpr int kFusedRowsF32 = 32 * kScoreThreads;
static int fused_f32_parts(const Shape& s) {
  const int64_t groups = (int64_t)s.B * s.Hkv;
  if (s.Lcap > kFusedRowsF32) return 0;
  const int64_t tiles = (s.cand_cap + 4 * kRowsPerWaveF32 - 1) / (4 * kRowsPerWaveF32);
  int64_t parts = (512 + groups - 1) / groups;
  parts = parts < tiles ? parts : tiles;
  return (int)(parts < 1 ? 1 : parts);
}
bool step_fuses_f32(const Shape& s) { return fused_f32_parts(s) > 0; }
hipError_t launch_candidates_score_f32(const Shape& s, const float* q, const KvView& kv, const int32_t* prev_topk, const int32_t* k,
                                       int32_t* cand, int32_t* cand_count, float* score, int64_t score_stride, int32_t* flags,
                                       hipStream_t st) {
  const int parts = fused_f32_parts(s);
  if (parts < 1) return hipErrorInvalidValue;
  const size_t lds = ((size_t)(s.Lcap + 31) / 32 + (s.cand_cap + parts - 1) / parts + kRowsPerWaveF32) * 4;
  const float scale = 0.08838834764831845f;   // 1/sqrt(128)
#define LFPS_LAUNCH_CSF(GG, PAGED)                                                                                              \
  hipLaunchKernelGGL((k_candidates_score_f32<GG, PAGED>), dim3(parts, s.B * s.Hkv), dim3(kScoreThreads), lds, st, s, q,          \
                     (const float*)kv.k, kv.stride_b, kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, prev_topk, k, cand,       \
                     cand_count, score, score_stride, scale, flags)
#define LFPS_LAUNCH_CSF_G(GG)                      \
  if (kv.page.table) LFPS_LAUNCH_CSF(GG, true);    \
  else LFPS_LAUNCH_CSF(GG, false)
  switch (s.G) {
    case 1: LFPS_LAUNCH_CSF_G(1); break;
    case 2: LFPS_LAUNCH_CSF_G(2); break;
    case 4: LFPS_LAUNCH_CSF_G(4); break;
    default: return hipErrorInvalidValue;
  }
#undef LFPS_LAUNCH_CSF_G
#undef LFPS_LAUNCH_CSF
  return hipGetLastError();
}

// Smallest part size in candidate slots, and the pieces a group can then be cut into (<= 1024).
int filter_min_seg_rows(const Shape& s) { return (((s.cand_cap + 999) / 1000) + 63) & ~63; }
int filter_nseg(const Shape& s) { return s.cand_cap / filter_min_seg_rows(s) + 2; }

template <int G, int kKind>
static hipError_t filter_resident_blocks(int out[2]) {
  int dev = 0;
  hipDeviceProp_t prop;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipGetDeviceProperties(&prop, dev);
  auto resident = [&](const void* kernel, int* n) {
    int per_cu = 0;
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kScoreThreads, 0);
    // two per CU is what the kernels are built for (__launch_bounds__); the FP8 variants would fit three,
    // measured slightly slower (smaller parts, no more bandwidth)
    if (per_cu > 2) per_cu = 2;
    *n = per_cu * prop.multiProcessorCount;
  };
  resident((const void*)k_filter_score_bf16<G, false, kKind, false>, &out[0]);
  resident((const void*)k_filter_score_bf16<G, true, kKind, false>, &out[1]);
  return e;
}

// Workgroups of the filtered scoring kernel that the current device holds at once (its launch size), for
// a contiguous cache (out[0]) and a paged one (out[1]); the variants differ in registers, hence in occupancy.
// k_kind: 0 bf16, 1 FP8, 2 fp16 keys.
hipError_t filter_score_blocks(const Shape& s, int k_kind, int out[2]) {
#define LFPS_RESIDENT(GG)                                                   \
  switch (k_kind) {                                                         \
    case kKindBf16: return filter_resident_blocks<GG, kKindBf16>(out);      \
    case kKindFp8: return filter_resident_blocks<GG, kKindFp8>(out);        \
    case kKindF16: return filter_resident_blocks<GG, kKindF16>(out);        \
    default: return hipErrorInvalidValue;                                   \
  }
  switch (s.G) {
    case 1: LFPS_RESIDENT(1)
    case 2: LFPS_RESIDENT(2)
    case 4: LFPS_RESIDENT(4)
    default: return hipErrorInvalidValue;
  }
#undef LFPS_RESIDENT
}

hipError_t launch_filter_score(const Shape& s, const float* q, const KvView& kv, const int32_t* cand,
                               const int32_t* cand_count, const int64_t* group_start, const int64_t* line_total,
                               const float* thr_state, float margin, float* tau_out, const int32_t* skip_if, float* score,
                               int32_t* slot_out, int64_t score_stride, int32_t* seg_count, int32_t* seg_rows_out,
                               int n_blocks, int32_t* flags, bool dense, int nseg, hipStream_t st) {
  if (n_blocks < 1) return hipErrorInvalidValue;
  const bool f16 = kv.f16;
  dim3 grid((unsigned)n_blocks), block(kScoreThreads);
  const float scale = 0.08838834764831845f;
#define LFPS_LAUNCH_FILTER_D(GG, PAGED, FP8, DENSE)                                                                \
  hipLaunchKernelGGL((k_filter_score_bf16<GG, PAGED, FP8, DENSE>), grid, block, 0, st, s, q, kv.k, kv.stride_b,    \
                     kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, cand, cand_count, group_start, line_total,    \
                     thr_state, margin, tau_out, skip_if, score, slot_out, score_stride, seg_count, seg_rows_out,                    \
                     filter_min_seg_rows(s), nseg, scale, flags)
#define LFPS_LAUNCH_FILTER_P(GG, PAGED, FP8)       \
  if (dense) {                                     \
    LFPS_LAUNCH_FILTER_D(GG, PAGED, FP8, true);    \
  } else {                                         \
    LFPS_LAUNCH_FILTER_D(GG, PAGED, FP8, false);   \
  }
#define LFPS_LAUNCH_FILTER(GG)                        \
  if (kv.page.table && kv.k_fp8) {                    \
    LFPS_LAUNCH_FILTER_P(GG, true, kKindFp8);         \
  } else if (kv.page.table && f16) {                  \
    LFPS_LAUNCH_FILTER_P(GG, true, kKindF16);         \
  } else if (kv.page.table) {                         \
    LFPS_LAUNCH_FILTER_P(GG, true, kKindBf16);        \
  } else if (kv.k_fp8) {                              \
    LFPS_LAUNCH_FILTER_P(GG, false, kKindFp8);        \
  } else if (f16) {                                   \
    LFPS_LAUNCH_FILTER_P(GG, false, kKindF16);        \
  } else {                                            \
    LFPS_LAUNCH_FILTER_P(GG, false, kKindBf16);       \
  }
  switch (s.G) {
    case 1: LFPS_LAUNCH_FILTER(1); break;
    case 2: LFPS_LAUNCH_FILTER(2); break;
    case 4: LFPS_LAUNCH_FILTER(4); break;
    default: return hipErrorInvalidValue;
  }
#undef LFPS_LAUNCH_FILTER_P
#undef LFPS_LAUNCH_FILTER_D
#undef LFPS_LAUNCH_FILTER
  return hipGetLastError();
}

hipError_t launch_head_score(const Shape& s, int dtype, const float* q, const KvView& kv, const int32_t* idx,
                             const int32_t* k, float* idx_score, hipStream_t st) {
  dim3 grid((s.kmax + 255) / 256, s.B * s.Hq), block(256);
  const float scale = 0.08838834764831845f;
#define LFPS_LAUNCH_HS(TYPE, PAGED)                                                                            \
  hipLaunchKernelGGL((k_head_score<TYPE, PAGED>), grid, block, 0, st, s, q, (const TYPE*)kv.k, kv.stride_b,     \
                     kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, idx, k, idx_score, scale)
  const bool paged = kv.page.table != nullptr;
  if (dtype == LFPS_BF16 && kv.k_fp8) {
    if (paged) LFPS_LAUNCH_HS(uint8_t, true);
    else LFPS_LAUNCH_HS(uint8_t, false);
  } else if (dtype == LFPS_BF16) {
    if (paged) LFPS_LAUNCH_HS(uint16_t, true);
    else LFPS_LAUNCH_HS(uint16_t, false);
  } else if (dtype == LFPS_F16) {
    if (paged) LFPS_LAUNCH_HS(_Float16, true);
    else LFPS_LAUNCH_HS(_Float16, false);
  } else {
    if (paged) LFPS_LAUNCH_HS(float, true);
    else LFPS_LAUNCH_HS(float, false);
  }
#undef LFPS_LAUNCH_HS
  return hipGetLastError();
}

}  // namespace lfps
