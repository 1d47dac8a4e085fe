// S1 + S2 of a chained step in one kernel, wide form: candidates from the Top-k rows of the step before and the filtered scores of
// their K rows, for contexts with more rows than the ranges of range_score.hip are for.
//
// Two workgroups per CU, two tiles per wave in flight; bound by the bytes of the rows and nearly as much by its instructions, about 400
// per tile.  A workgroup has two strips of its group's rows, half the request apart (wide_cut.h).  It marks the candidates among them in
// an LDS bitmap, and its waves take a quarter of those of either strip each.  The candidates are not listed: a wave expands the bitmap from
// where its quarter begins, 256 positions at a time, into a ring of its own.  What it leaves is what the range kernel does, with a strip for
// a range: survivors per head and (strip, wave) piece, ascending in position, the counts of every piece, and the bitmap.
//
// Why one kernel: against a kernel that lists the candidates of a group in memory and one that reads them back in equal parts, a step of
// 64 groups x 32K rows: 7.9 + 36.2 us and a boundary -> 40; of 128 x 128K 13.1 + 174 -> 172, of FP8 128 x 64K pages 9.6 + 47.4 -> 53.
// With four workgroups per CU and one tile each, 911 us for four steps of 128 x 128K instead of 810 (884 separately).
// Why two strips: Top-k rows crowd, and of rows in one piece either all or none are candidates then.  Four steps with the Top-k in the
// last eighth (quarter) of the rows, separate kernels -> one piece -> two strips: 64 groups x 32K rows 172 (212) -> 225 (226) -> 147
// (178), 16 x 128K 178 (206) -> 222 (217) -> 150 (178), 128 x 128K 625 (940) -> 915 (1465) -> 692 (870), 256 x 64K 630 (940) -> 630 (980)
// -> 570 (843).  Spread rows pay 2 to 4 % for it (the select finds twice the pieces), up to 6 % where a workgroup has few (four steps of 152 x
// 10072, separate kernels 148, one piece 110, two strips 117).  With four or eight strips the waves' quarters become
// short and the pieces many: 64 x 32K 43 and 45 us here and 15.0 and 16.0 in the select, instead of 40 and 14.6.
#include "candidates.h"
#include "range_geometry.h"
#include "range_rule.h"
#include "score_mfma.h"

namespace lfps {

constexpr int kWideStage = 256;        // survivors a wave holds per head before it writes them out
constexpr int kWideRing = 512;         // candidates of a wave, expanded
constexpr int kWideSpare = 16;

// K rows that the candidates of a request of n rows and budget k are, about: windows of 2 r + 2 rows around the Top-k rows of a group's
// heads, which have a part of them in common, and the recent rows and sinks.  How many workgroups a request gets hangs on it, and whether
// rows are read past the caches.
__device__ __forceinline__ float candidate_rows(const Shape& s, int n, int k) {
  const float heads = s.G == 4 ? 1.6f : (s.G == 2 ? 1.3f : 1.f), window = heads * (2.f * (float)s.radius + 2.f);
  const float nf = (float)(n < 1 ? 1 : (n > s.Lcap ? s.Lcap : n)), kf = (float)(k < 0 ? 0 : (k > s.kmax ? s.kmax : k));
  const float others = nf - (float)s.n_recent - (float)s.n_sink;
  return nf - (others > 0.f ? others : 0.f) * __expf(-window * kf / nf);
}

// may_once: the candidates may take more than the memory-side cache holds; rows are then read past it, see k_filter_score_bf16.
template <int G, bool kPaged, int kKind>
__global__ __launch_bounds__(kScoreThreads, 2) void k_wide_score(
    Shape s, const float* __restrict__ q, const void* __restrict__ K, int64_t stride_b, int64_t stride_h,
    int64_t stride_n, KvPage page, const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ prev_topk,
    const int32_t* __restrict__ kk, const float* __restrict__ thr_state, float margin, float* __restrict__ tau_out,
    const int32_t* __restrict__ skip_if, float* __restrict__ score, int32_t* __restrict__ slot_out,
    int64_t score_stride, int32_t* __restrict__ seg_count, int nseg, int32_t* __restrict__ parts_out, uint32_t* __restrict__ bitmap,
    int bitmap_words, WidePlan plan, float scale, int32_t* __restrict__ flags, int may_once) {
  __shared__ float stage_score[4][G][kWideStage];
  __shared__ uint16_t stage_place[4][G][kWideStage];
  __shared__ u32x4 turn[4][StreamTile<kKind>::kLdsChunks];
  __shared__ uint16_t ring[4][kWideRing];
  extern __shared__ uint32_t bm[];                        // the workgroup's places, and kWideSpare words that expanding may read
  request_arguments<decltype(&k_wide_score<G, kPaged, kKind>)>();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, kb = lane >> 4;
  const WideBlock at_block(s.B * s.Hkv, s.Hkv, gridDim.x, gridDim.y, blockIdx.x, blockIdx.y, blockIdx.z);
  const bool extra = at_block.extra;
  int b = at_block.b;
  const int g = at_block.g;

  using Rows = RowMap<kPaged>;
  using Tile = StreamTile<kKind>;
  using Op = typename Tile::Operand;

  // ---- what the workgroup needs is requested before anything is waited for
  // The entries tid, tid + 256, ... of every head's Top-k row, eight at a time, as in the range kernel.
  // Before them the lengths and budgets of the first 64 requests, one to a lane.
  const bool weigh = plan.slots > 0 || may_once;
  const int b_lane = lane < s.B ? lane : 0;
  int n_lane = 0, k_lane = 0;
  if (weigh) {
    n_lane = seq_lens[b_lane];
    k_lane = kk[b_lane];
  }
  constexpr int kEach = 8;
  int ids[kEach][G];
  const int32_t* pt;
  auto fetch = [&](int j0) {
#pragma unroll
    for (int u = 0; u < kEach; ++u) {
      const int at = j0 + kScoreThreads * u;
      if (at >= s.kmax) break;                             // (uniform)
#pragma unroll
      for (int h = 0; h < G; ++h) ids[u][h] = (pt + (int64_t)h * s.kmax)[at + tid < s.kmax ? at + tid : s.kmax - 1];
    }
  };
  int n, k_raw;
  auto ask_for = [&](int request) {
    pt = prev_topk + ((int64_t)request * s.Hq + (int64_t)g * G) * s.kmax;
    fetch(0);
    n = seq_lens[request];
    k_raw = kk[request];
    asm volatile("" ::"s"(n), "s"(k_raw));                 // (beside the entries)
  };
  ask_for(b);

  // ---- whose rows: part `part` of `parts` of request b
  int parts = plan.parts, part = at_block.part;
  float all_rows = 0.f;
  if (weigh && s.B <= 64 && !__ballot(n_lane != n || k_lane != k_raw)) {      // (all alike: 0.5 us for a step of 144 groups)
    if (extra) return;
    all_rows = (float)s.B * candidate_rows(s, n, k_raw);
  } else if (weigh) {
    auto length = [&](int request) {
      const int of = request < 64 ? n_lane : seq_lens[request < s.B ? request : 0];
      return of < 0 ? 0 : (of > s.Lcap ? s.Lcap : of);
    };
    auto rows_of = [&](int request) { return candidate_rows(s, length(request), request < 64 ? k_lane : kk[request < s.B ? request : 0]); };
    float largest = 0.f;
    int fewest = 0;
    for (int c0 = 0; c0 < s.B; c0 += 64) {
      const bool is = c0 + lane < s.B;
      const float rows = is ? rows_of(c0 + lane) : 0.f;
      all_rows += rows;
      largest = fmaxf(largest, rows);
      fewest += is ? fewest_parts(length(c0 + lane)) : 0;
    }
    all_rows = row16_sum(all_rows);
    all_rows += __shfl_xor(all_rows, 16);
    all_rows += __shfl_xor(all_rows, 32);
    all_rows = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(all_rows)));
    largest = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_max_in_last(largest)), 63));
    if (plan.slots > 0 && uneven(largest, all_rows, s.B)) {
      const int spare = plan.slots - __builtin_amdgcn_readlane(wave_inclusive_sum(fewest), 63);
      int slot = at_block.slot(s.B, s.Hkv, parts);
      parts = 0;
      for (int c0 = 0; c0 < s.B; c0 += 64) {               // (every wave of every workgroup finds the same numbers)
        const int mine = c0 + lane < s.B ? parts_of_request(length(c0 + lane), rows_of(c0 + lane), all_rows, spare, plan.most) : 0;
        const int upto = wave_inclusive_sum(mine), total = __builtin_amdgcn_readlane(upto, 63);
        if (slot < total) {
          const int at = __builtin_ctzll(__ballot(slot < upto));
          b = c0 + at;
          parts = __builtin_amdgcn_readlane(mine, at);
          part = slot - (__builtin_amdgcn_readlane(upto, at) - parts);
          break;
        }
        slot -= total;
      }
      if (parts == 0) return;
      ask_for(b);
    } else if (extra) {
      return;
    }
  } else if (extra) {
    return;
  }
  const int bg = b * s.Hkv + g;
  const int64_t head0 = (int64_t)b * s.Hq + (int64_t)g * G, my_head = head0 + (kb < G ? kb : 0);
  const float thr = thr_state[my_head];
  const int skip_word = *(skip_if ? skip_if + my_head : seq_lens);             // (no gate: any word)
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const Strips mine(n, parts, part);                      // (of the request's rows, not of the context's)
  if (mine.first >= n) return;                            // (nobody reads the piece counts of such a strip)
  const int strip_words = mine.rows >> 5;
  for (int w = tid; w < 2 * strip_words; w += kScoreThreads) bm[w] = 0u;
  const int r = s.radius;
  Op A[4];
  QueryRows query;                                         // split behind the requests for the first rows
  query.load(q, head0, G, j, kb);
  const bool once = may_once && all_rows * (float)s.Hkv * (float)(kD * Tile::kElemBytes) > (float)kKeptBytes;
  __syncthreads();

  // ---- S1: my candidates as a bitmap of places
  const int k = k_raw < 0 ? 0 : (k_raw > s.kmax ? s.kmax : k_raw);
  const int rc = r < s.Lcap ? r : s.Lcap;                  // (no sum overflows)
  // (The strips of a group's only workgroup follow on each other: one of twice their length.  A window of at most 32 rows touches one
  // strip, then: two are at least 64 rows apart.  Longer windows read the entries again: among the unrolled ones they made 16 KB more code,
  // and two kernels in turn share the instruction cache: four steps of 8 x 32K 230.5 -> 228.8 us, of 16 x 128K 826 -> 818.)
  const StripWindows one(n, mine.first, parts == 1 ? 2 * mine.rows : mine.rows, rc), two(n, parts == 1 ? n : mine.second, mine.rows, rc);
  if (rc <= kWindowRadius) {
    for (int j0 = 0;;) {
#pragma unroll
      for (int u = 0; u < kEach; ++u) {
        const int at = j0 + kScoreThreads * u;
        if (at >= k) break;                                // (uniform)
#pragma unroll
        for (int h = 0; h < G; ++h) {
          const int e = ids[u][h];
          const bool in_two = two.touches(e);
          if (at + tid < k && (in_two || one.touches(e))) {
            const int begin = in_two ? two.begin : one.begin, end = in_two ? two.end : one.end;
            set_bit_window(bm + (in_two ? strip_words : 0), StripWindows::from(e, rc, begin), StripWindows::to(e, rc, begin, end));
          }
        }
      }
      j0 += kScoreThreads * kEach;
      if (j0 >= k) break;
      fetch(j0);
    }
  } else {
    for (int at = tid; at < k; at += kScoreThreads) {
      int e[G];
#pragma unroll
      for (int h = 0; h < G; ++h) e[h] = pt[(int64_t)h * s.kmax + at];
#pragma unroll
      for (int h = 0; h < G; ++h) {
        if (one.touches(e[h])) set_bit_range(bm, StripWindows::from(e[h], rc, one.begin), StripWindows::to(e[h], rc, one.begin, one.end));
        if (two.touches(e[h]))
          set_bit_range(bm + strip_words, StripWindows::from(e[h], rc, two.begin), StripWindows::to(e[h], rc, two.begin, two.end));
      }
    }
  }
  if (tid < 2) {                                           // recent rows and sinks
    const int from = tid ? mine.second : mine.first, to = n - from < mine.rows ? n : from + mine.rows, place = tid * mine.rows - from;
    if (from < n) {
      const int recent = n - s.n_recent > from ? n - s.n_recent : from, sinks = s.n_sink < to ? s.n_sink : to;
      if (recent < to) set_bit_range(bm, place + recent, place + to - 1);
      if (sinks > from) set_bit_range(bm, place + from, place + sinks - 1);
    }
  }
  __syncthreads();

  // ---- S2: the pieces of this wave: of either strip the candidates [wave * per, (wave + 1) * per), per = a quarter of them.  Every wave
  // counts for itself; it needs the place of its first candidate.
  struct Piece {
    int count, place;
  } piece[2];
  {
    const int own = (strip_words + 63) >> 6, w0 = lane * own;
    int here[2] = {0, 0}, upto[2], at[2], begin[2], word[2], in_word[2], left[2];
#pragma unroll
    for (int u = 0; u < kWideMax / 2 / 32 / 64; ++u) {
      if (u >= own) break;                                 // (uniform)
#pragma unroll
      for (int x = 0; x < 2; ++x) here[x] += w0 + u < strip_words ? __popc(bm[x * strip_words + w0 + u]) : 0;
    }
#pragma unroll
    for (int x = 0; x < 2; ++x) {                          // the lane of my first candidate
      upto[x] = wave_inclusive_sum(here[x]);
      const int total = __builtin_amdgcn_readlane(upto[x], 63), per = (total + 3) >> 2, mine_left = total - wave * per;
      piece[x].count = mine_left < per ? (mine_left > 0 ? mine_left : 0) : per;
      begin[x] = wave * per;
      at[x] = __builtin_ctzll(__ballot(begin[x] < upto[x]) | 1ull << 63);
      const int w = at[x] * own + lane;
      word[x] = lane < own && w < strip_words ? (int)bm[x * strip_words + w] : 0;
    }
#pragma unroll
    for (int x = 0; x < 2; ++x) {                          // its word,
      in_word[x] = __popc((uint32_t)word[x]);
      left[x] = begin[x] - __builtin_amdgcn_readlane(upto[x] - here[x], at[x]);
      const int upto_word = wave_inclusive_sum(in_word[x]);
      const int lane_of = __builtin_ctzll(__ballot(left[x] < upto_word) | 1ull << 63);
      left[x] -= __builtin_amdgcn_readlane(upto_word - in_word[x], lane_of);
      piece[x].place = 32 * (x * strip_words + at[x] * own + lane_of);
      word[x] = __builtin_amdgcn_readlane(word[x], lane_of);
    }
#pragma unroll
    for (int x = 0; x < 2; ++x) {                          // and its bit
      const uint32_t bits = (uint32_t)word[x], bit = lane & 31;
      piece[x].place += __builtin_ctzll(__ballot((bits >> bit & 1u) && __popc(bits & ((1u << bit) - 1u)) == left[x]) | 1ull << 63);
    }
  }
  const Piece a = piece[0], z = piece[1];                  // (places of empty pieces are not used)
  const int cnt = a.count + z.count;
  const RangePieces geo(n, 0, 2 * parts);
  const int piece_a = 4 * part + wave, piece_z = 4 * (parts + part) + wave;
  const bool skipped = skip_if && skip_word != 0;         // bypassed head: nothing is kept for it
  const uint64_t nans = __ballot(kb < G && isnan(thr) && !skipped);
  auto leave = [&](int kept_a, int kept) {                 // (no store before the last load: a wait for that would wait for the store)
    for (int w = tid; w < 2 * strip_words; w += kScoreThreads) {
      const int to = mine.row_of(32 * w) >> 5;
      if (to < bitmap_words) bitmap[(int64_t)bg * bitmap_words + to] = bm[w];
    }
    if (j < 2 && kb < G && (j == 0 || mine.second < n))
      seg_count[my_head * nseg + (j == 0 ? piece_a : piece_z)] = j == 0 ? a.count << 16 | kept_a : z.count << 16 | (kept - kept_a);
    if (j == 0 && kb < G && piece_a == 0) tau_out[my_head] = thr - margin;
    if (lane == 0 && piece_a == 0) parts_out[bg] = parts;
  };
  if (cnt == 0 || nans) {
    leave(0, 0);
    return;
  }
  const float tau = kb < G && !skipped ? thr - margin : INFINITY;
  const uint32_t below = (1u << j) - 1u;                 // lanes of my 16-lane group with a lower row
  float* st_s = stage_score[wave][kb < G ? kb : 0];
  uint16_t* st_i = stage_place[wave][kb < G ? kb : 0];
  constexpr int ES = Tile::kElemBytes, T = kRowsPerWaveIter;
  const char* Kbg = static_cast<const char*>(K) + Rows::base(b, g, stride_b, stride_h) * ES;
  int run = 0, staged = 0;                               // my head's survivors in global memory, and waiting in LDS
  int kept_a = 0;                                        // of both, in the first strip (once its last candidate is scored)

  // (survivors are staged so that the loop holds no global store: a wait for a load would wait for those before it)
  const int out_a = geo.start(piece_a), out_z = mine.second < n ? geo.start(piece_z) : 0;
  auto flush = [&]() {
    wave_lds_order();
    if (kb < G) {                                         // sixteen lanes write for a head
      float* dsc = score + my_head * score_stride + run;
      int32_t* dsl = slot_out + my_head * score_stride + run;
      for (int e = j; e < staged; e += 16) {
        const int place = st_i[e], to = place < mine.rows ? out_a + e : out_z + e - kept_a;
        dsc[to] = st_s[e];
        dsl[to] = mine.row_of(place);
      }
    }
    run += staged;
    staged = 0;
    wave_lds_order();
  };
  // Candidates e0 + lane of mine (past the end: the last one, never kept), as places.  The ring is filled from place `from` on, the
  // first strip's, then the second's; what comes behind a piece's last candidate is overwritten.
  int from = a.place, filled = 0;
  bool second = false;
  auto ids_of = [&](int e0) {
    const int e = e0 + lane < cnt ? e0 + lane : cnt - 1;
    const int need = e0 + T < cnt ? e0 + T : cnt;
    uint16_t* to_ring = ring[wave];
    wave_lds_order();
    while (filled < need) {                               // (ends: the pieces hold their counts from their first places on)
      if (!second && filled >= a.count) {
        second = true;
        from = z.place;
      }
      const int place = from + 4 * lane, w = place >> 5;
      const uint32_t four = __builtin_amdgcn_alignbit(bm[w + 1], bm[w], place & 31) & 15u;
      const int here = __popc(four), upto = wave_inclusive_sum(here);
      int to = filled + upto - here;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (four >> c & 1u) to_ring[to & (kWideRing - 1)] = (uint16_t)(place + c);
        to += four >> c & 1u;
      }
      filled += __builtin_amdgcn_readlane(upto, 63);
      if (!second && filled > a.count) filled = a.count;
      from += 256;
      if (from >= 64 * strip_words) {                     // (a piece that holds its count is expanded by then)
        if (second) break;
        filled = a.count;
      }
    }
    wave_lds_order();
    return (int)to_ring[e & (kWideRing - 1)];
  };
  auto consume = [&](const Tile& Bt, int ids, int e0) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const KSub<kKind> sub = Bt.sub(t, turn[wave], lane);
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) acc = mfma16(A[kk], sub.operand(kk), acc);
      const float v = Split3<Op>::sum(acc) * scale;
      const bool pass = kb < G && e0 + 16 * t + j < cnt && v >= tau;
      const uint32_t gm = (uint32_t)(__ballot(pass) >> (16 * kb)) & 0xFFFFu;   // my head's 16 rows
      const int place = lane_value(ids, j, 16 * t);
      if (pass) {
        const int o = staged + __popc(gm & below);
        st_s[o] = v;
        st_i[o] = (uint16_t)place;
      }
      const int of_a = a.count - (e0 + 16 * t);            // (uniform) of these sixteen and behind
      if (of_a > 0 && of_a <= 16) kept_a = run + staged + __popc(gm & ((1u << of_a) - 1u));
      staged += __popc(gm);
    }
    if (__ballot(staged > kWideStage - T)) flush();      // no room for one more tile
  };
  // Paged cache: the block-table lookup of the next tile is issued before the loads of this one, so that the wait for it
  // does not wait for them (memory operations complete in order).
  auto lookup = [&](int id) { return Rows::phys(page, b, mine.row_of(id)); };
  int id = ids_of(0);                                     // of the next tile
  int phys = lookup(id);
  auto request = [&](Tile& Bt, int& in_flight, int e0) {
    const int phys_now = phys;
    in_flight = id;
    id = ids_of(e0 + T);
    if constexpr (kPaged) {
      asm volatile("" ::"v"(phys_now));
      phys = lookup(id);
      __builtin_amdgcn_sched_barrier(0);
    } else {
      phys = lookup(id);
    }
    Bt.fetch(Kbg, phys_now, lane, [&](int p) { return Rows::offset(page, p, stride_b, stride_n) * ES; }, once);
  };
  Tile B0, B1;
  int f0, f1, e0 = 0;
  request(B0, f0, 0);
  __builtin_amdgcn_sched_barrier(0);
  report_q_range(query.operand(A, G, j), flags);
  for (; e0 + 2 * T < cnt; e0 += 2 * T) {
    request(B1, f1, e0 + T);
    consume(B0, f0, e0);
    request(B0, f0, e0 + 2 * T);
    consume(B1, f1, e0 + T);
  }
  if (e0 + T < cnt) {
    request(B1, f1, e0 + T);
    consume(B0, f0, e0);
    consume(B1, f1, e0 + T);
  } else {
    consume(B0, f0, e0);
  }
  flush();
  leave(kept_a, run);
}

// ----------------------------------------------------------------------------- launcher
WidePlan wide_plan(const Shape& s) {
  const int64_t groups = (int64_t)s.B * s.Hkv;
  if (range_rows_for(groups, s.Lcap, s.G, false)) return WidePlan{0, 0, 0, 0};
  Shape dense = s;                                          // (the counts of the exact Top-k, which has all rows for candidates)
  dense.cand_cap = s.Lcap;
  return wide_plan_for(s.B, s.Hkv, s.Lcap, filter_nseg(dense));
}

template <int G, bool kPaged, int kKind>
static constexpr auto wide_kernel = &k_wide_score<G, kPaged, kKind>;

hipError_t launch_wide_score(const Shape& s, const float* q, const KvView& kv, const int32_t* prev_topk, const int32_t* k,
                             const float* thr_state, float margin, float* tau_out, const int32_t* skip_if, float* score, int32_t* slot_out,
                             int64_t score_stride, int32_t* seg_count, int nseg, int32_t* parts_of, uint32_t* bitmap, int bitmap_words,
                             int32_t* flags, hipStream_t st) {
  const int groups = s.B * s.Hkv;
  const int kind = kv.k_fp8 ? kKindFp8 : (kv.f16 ? kKindF16 : kKindBf16);
  const bool paged = kv.page.table != nullptr;
  const WidePlan plan = wide_plan(s);
  if (plan.rows <= 0) return hipErrorInvalidValue;
  // (cand_cap is at least what the windows can cover)
  const int may_once = (int64_t)groups * s.cand_cap * kD * (kind == kKindFp8 ? 1 : 2) > kKeptBytes;
  const WideGrid grid = wide_grid(plan, s.B, s.Hkv);
  hipError_t e = hipErrorInvalidValue;
  auto launch = [&](auto heads, auto pages, auto form) {
    constexpr int G = decltype(heads)::value, kKind = decltype(form)::value;
    constexpr bool kPaged = decltype(pages)::value;
    if (s.G != G || paged != kPaged || kind != kKind) return;
    hipLaunchKernelGGL((wide_kernel<G, kPaged, kKind>), dim3(grid.beside, grid.parts, grid.deep), dim3(kScoreThreads),
                       (size_t)(plan.slots ? kWideMax : plan.rows) / 8 + kWideSpare * 4, st, s, q, kv.k, kv.stride_b, kv.stride_h,
                       kv.stride_n, kv.page, kv.seq_lens, prev_topk, k, thr_state, margin, tau_out, skip_if, score, slot_out, score_stride, seg_count, nseg, parts_of, bitmap, bitmap_words, plan,
                       0.08838834764831845f /* 1/sqrt(128) */, flags, may_once);
    e = hipGetLastError();
  };
  auto of_kinds = [&](auto heads, auto pages) {
    launch(heads, pages, std::integral_constant<int, kKindBf16>{});
    launch(heads, pages, std::integral_constant<int, kKindFp8>{});
    launch(heads, pages, std::integral_constant<int, kKindF16>{});
  };
  auto of_heads = [&](auto heads) {
    of_kinds(heads, std::false_type{});
    of_kinds(heads, std::true_type{});
  };
  of_heads(std::integral_constant<int, 1>{});
  of_heads(std::integral_constant<int, 2>{});
  of_heads(std::integral_constant<int, 4>{});
  return e;
}

}  // namespace lfps
