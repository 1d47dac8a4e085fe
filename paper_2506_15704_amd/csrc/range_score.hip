// S1 + S2 of a chained step in one kernel: the candidates of a KV group (Alg. 1 lines 6-7; Eq. 7 and 9) and the filtered
// scores of their rows (Alg. 1 line 8), for 16-bit and FP8 keys.
//
// The positions of a group are cut into ranges of `range` rows, one per workgroup.  A workgroup marks its range's
// candidates in an LDS bitmap (from the Top-k rows of the step before, of which it keeps what touches its range, or from
// the flag words of the table scan), lists them in LDS and scores their K rows at once, the list in four equal pieces,
// one per wave.  What reaches a head's threshold (the k-th best score of the step before minus a margin; NaN: no step
// before, nothing is kept and the select takes its unfiltered pass) goes to the head's score / position rows, ascending
// in position, with the numbers of survivors and candidates of every piece in seg_count.  The bitmap goes to memory too,
// for the heads that need that unfiltered pass.
//
// Larger contexts from the Top-k take the wide form, a kernel of its own (wide_score.hip).
//
// Why one kernel: as two, a step of 8 groups x 32K rows spent 7.8 + 14.5 us here, of which the rows themselves are 5 us;
// the rest is two launches and the round trips
// candidates -> list -> geometry -> list -> rows.  Together: 13.7 us, 12.2 with the rows through LDS:
// every load instruction covers whole rows (StreamTile, here with ordinary loads; 16-bit keys).  With a lane's own 64 bytes of a row in four
// loads, each of these touches 32 cache lines instead of 8, and with one tile per wave and eight to sixteen waves per CU all asking at
// once the address unit was what the first rows waited for.  11.4 us with the entries of a Top-k row strided over the lanes and the
// survivors of all heads written side by side, 9.2 with length and budget asked for beside the Top-k entries.  (A stage of 160 survivors makes room for it at four workgroups per CU.)
#include "candidates.h"
#include "range_geometry.h"
#include "score_mfma.h"

namespace lfps {

constexpr int kRangeStage = 160;        // survivors a wave holds per head before it writes them out

template <int G, bool kPaged, int kKind, bool kTables>
__global__ __launch_bounds__(kScoreThreads, 4) void k_range_score(
    Shape s, const float* __restrict__ q, const void* __restrict__ K, int64_t stride_b, int64_t stride_h,
    int64_t stride_n, KvPage page, const int32_t* __restrict__ seq_lens, RangeSource from, const int32_t* __restrict__ kk,
    const float* __restrict__ thr_state, float margin, float* __restrict__ tau_out, const int32_t* __restrict__ skip_if,
    float* __restrict__ score, int32_t* __restrict__ slot_out,
    int64_t score_stride, int32_t* __restrict__ seg_count, int nseg, uint32_t* __restrict__ bitmap, int bitmap_words,
    int range, float scale, int32_t* __restrict__ flags) {
  __shared__ float stage_score[4][G][kRangeStage];
  __shared__ uint16_t stage_slot[4][G][kRangeStage];          // relative to the range's first row
  __shared__ u32x4 turn[4][kKind == kKindFp8 ? 1 : StreamTile<kKind>::kLdsChunks];
  __shared__ uint32_t bm[kRangeMax / 32];
  __shared__ int wave_tot[4];
  extern __shared__ uint16_t list[];                     // the range's candidates, relative to its first row
  request_arguments<decltype(&k_range_score<G, kPaged, kKind, kTables>)>();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, kb = lane >> 4;
  // grid (8 groups side by side, ranges, the other groups): workgroups are dealt to the XCDs in turn, and those of a group share an L2
  const int bg = blockIdx.z * gridDim.x + blockIdx.x, b = (int)((uint32_t)bg / (uint32_t)s.Hkv), g = bg - b * s.Hkv;

  using Rows = RowMap<kPaged>;
  // (FP8 rows, a line each, come in two loads of a lane's own bytes: four steps of 1 x 32K, k = 400 71.4 -> 69.0 us, of 8 x 16000 110.6 ->
  // 106.7; with the cache in host memory 1288 -> 1126.)
  using Tile = std::conditional_t<kKind == kKindFp8, KTile<kKind>, StreamTile<kKind>>;
  using Op = typename Tile::Operand;

  // ---- what the workgroup needs is requested before anything is waited for
  // The entries tid, tid + 256, ... of every head's Top-k row, eight at a time.  (Neighbouring lanes hold neighbouring entries: the few
  // that touch the range stand side by side in a list that ascends, and one pass of one wave marks them.  Four entries a lane made
  // that wave take sixteen passes in turn: 8 groups x 32K rows, 2.0 us here instead of 1.1.)
  constexpr int kEach = kTables ? 1 : 8;
  int ids[kEach][G];
  const int32_t* pt = kTables ? nullptr : from.prev_topk + ((int64_t)b * s.Hq + (int64_t)g * G) * s.kmax;
  auto fetch = [&](int j0) {
    if constexpr (!kTables) {
#pragma unroll
      for (int u = 0; u < kEach; ++u) {
        const int at = j0 + kScoreThreads * u;
        if (at >= s.kmax) break;                           // (uniform)
#pragma unroll
        for (int h = 0; h < G; ++h) ids[u][h] = (pt + (int64_t)h * s.kmax)[at + tid < s.kmax ? at + tid : s.kmax - 1];
      }
    }
  };
  fetch(0);
  int n = seq_lens[b];
  const int k_raw = kTables ? 0 : kk[b];
  // (Scalar loads beside the entries.  Behind them, the budget as a vector load, each was a trip to memory of its own.)
  asm volatile("" ::"s"(n), "s"(k_raw));
  const int64_t head0 = (int64_t)b * s.Hq + (int64_t)g * G, my_head = head0 + (kb < G ? kb : 0);
  const float thr = thr_state[my_head];
  const int skip_word = *(skip_if ? skip_if + my_head : seq_lens);             // (no gate: any word)
  const int words = range >> 5;
  if (tid < words) bm[tid] = 0u;
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const int lo = blockIdx.y * range;
  if (lo >= n) return;                                   // (nobody reads the piece counts of such a range)
  const int hi = n - lo < range ? n : lo + range;
  const int r = s.radius;
  // The query is split behind the requests for the first rows, beside their latency (four steps of 8 groups x 32K rows 105.7 ->
  // 103.3 us, of 32 x 12K FP8 88.8 -> 88.1), where the registers allow it: not of fp16, whose split takes the most of them (beside a
  // tile it spills), and not of paged rows (8 x 32K 114.4 -> 116.1).
  constexpr bool kSplitLate = !Split3<Op>::kHalf && !kPaged;
  Op A[4];
  QueryRows query;
  query.load(q, head0, G, j, kb);
  if constexpr (!kSplitLate) report_q_range(query.operand(A, G, j), flags);
  __syncthreads();

  // ---- S1: the candidates of [lo, hi) as a bitmap
  if constexpr (kTables) {
    const int w = (lo >> 5) + tid, W = (n + 31) >> 5;
    if (tid < words && w < W) {
      uint32_t before[G], mid[G], after[G], mean[G];
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const int64_t row = (head0 + h) * from.flag_words;
        before[h] = from.f0[row + (w > 0 ? w - 1 : 0)];
        mid[h] = from.f0[row + w];
        after[h] = from.f0[row + (w + 1 < W ? w + 1 : w)];
        mean[h] = from.fm[row + w];
      }
#pragma unroll
      for (int h = 0; h < G; ++h) {
        before[h] = w > 0 ? before[h] : 0u;
        after[h] = w + 1 < W ? after[h] : 0u;
      }
      uint32_t acc = 0u;
#pragma unroll
      for (int h = 0; h < G; ++h) acc |= widen_word(before[h], mid[h], after[h], r) & mean[h];
      bm[tid] = acc;
    }
    __syncthreads();
  } else {
    const int k = k_raw < 0 ? 0 : (k_raw > s.kmax ? s.kmax : k_raw);
    // an entry i touches [lo, hi) with its window [i - r, i + r + 1] when first <= i <= last (r capped: no sum overflows)
    const int rc = r < s.Lcap ? r : s.Lcap;
    const int first = lo - 1 - rc > 0 ? lo - 1 - rc : 0, last = hi - 1 + rc < n - 1 ? hi - 1 + rc : n - 1;
    const uint32_t width = (uint32_t)(last - first);
    for (int j0 = 0;;) {
#pragma unroll
      for (int u = 0; u < kEach; ++u) {
        const int at = j0 + kScoreThreads * u;
        if (at >= k) break;                                // (uniform)
#pragma unroll
        for (int h = 0; h < G; ++h) {
          const int e = ids[u][h];
          if ((uint32_t)(e - first) <= width && at + tid < k) {
            const int a = e - rc - lo, z = e + rc + 1 - lo;
            if (rc <= kWindowRadius) set_bit_window(bm, a < 0 ? 0 : a, z < hi - lo ? z : hi - 1 - lo);
            else set_bit_range(bm, a < 0 ? 0 : a, z < hi - lo ? z : hi - 1 - lo);
          }
        }
      }
      j0 += kScoreThreads * kEach;
      if (j0 >= k) break;
      fetch(j0);
    }
  }
  if (tid == 0) {
    const int first = n - s.n_recent < lo ? lo : n - s.n_recent;
    if (first < hi) set_bit_range(bm, first - lo, hi - 1 - lo);
    const int sinks = s.n_sink < hi ? s.n_sink : hi;
    if (sinks > lo) set_bit_range(bm, 0, sinks - 1 - lo);
  }
  __syncthreads();

  // ---- the list: thread t owns the bits [t * nb, (t + 1) * nb), nb = the power of two that 256 threads cover the range with
  const int nb = range <= kScoreThreads ? 1 : 1 << (32 - __builtin_clz((uint32_t)(range - 1) / kScoreThreads)), bit0 = tid * nb;
  uint32_t bits = bit0 < range ? (bm[bit0 >> 5] >> (bit0 & 31)) & (nb == 32 ? 0xFFFFFFFFu : (1u << nb) - 1u) : 0u;
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
  while (bits) {
    list[at++] = (uint16_t)(bit0 + __ffs(bits) - 1);
    bits &= bits - 1;
  }
  __syncthreads();

  // ---- S2: the piece of this wave, entries [c0, c0 + cnt) of the list
  const RangePieces geo(n, range, 0);
  const int per = (((total + 3) >> 2) + 15) & ~15;
  const int c0 = wave * per;
  const int cnt = __builtin_amdgcn_readfirstlane(total - c0 < per ? (total - c0 > 0 ? total - c0 : 0) : per);
  const int piece = 4 * (int)blockIdx.y + wave;
  const int out0 = geo.start(piece);                      // where its survivors go in the heads' rows
  const bool skipped = skip_if && skip_word != 0;         // bypassed head: nothing is kept for it
  const uint64_t nans = __ballot(kb < G && isnan(thr) && !skipped);
  auto leave = [&](int kept) {                           // (no store before the last load: a wait for that would wait for the store)
    if (tid < words && (lo >> 5) + tid < bitmap_words) bitmap[(int64_t)bg * bitmap_words + (lo >> 5) + tid] = bm[tid];
    if (j == 0 && kb < G) {
      seg_count[my_head * nseg + piece] = cnt << 16 | kept;
      if (piece == 0) tau_out[my_head] = thr - margin;
    }
  };
  if (cnt == 0 || nans) {
    leave(0);
    return;
  }
  const float tau = kb < G && !skipped ? thr - margin : INFINITY;
  const uint32_t below = (1u << j) - 1u;                 // lanes of my 16-lane group with a lower row
  float* st_s = stage_score[wave][kb < G ? kb : 0];
  uint16_t* st_i = stage_slot[wave][kb < G ? kb : 0];
  constexpr int ES = Tile::kElemBytes, T = kRowsPerWaveIter;
  const char* Kbg = static_cast<const char*>(K) + Rows::base(b, g, stride_b, stride_h) * ES;
  int run = 0, staged = 0;                               // my head's survivors in global memory, and waiting in LDS

  // (survivors are staged so that the loop holds no global store: a wait for a load would wait for those before it)
  auto flush = [&]() {
    wave_lds_order();
    if (kb < G) {                                         // sixteen lanes write for a head
      float* dsc = score + my_head * score_stride + out0 + run;
      int32_t* dsl = slot_out + my_head * score_stride + out0 + run;
      for (int e = j; e < staged; e += 16) {
        dsc[e] = st_s[e];
        dsl[e] = lo + st_i[e];
      }
    }
    run += staged;
    staged = 0;
    wave_lds_order();
  };
  // list entry e0 + lane (past the end: the last one, never kept), relative to the range
  auto ids_of = [&](int e0) { return (int)list[c0 + (e0 + lane < cnt ? e0 + lane : cnt - 1)]; };
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
      const int row = lane_value(ids, j, 16 * t);
      if (pass) {
        const int o = staged + __popc(gm & below);
        st_s[o] = v;
        st_i[o] = (uint16_t)row;
      }
      staged += __popc(gm);
    }
    if (__ballot(staged > kRangeStage - T)) flush();      // no room for one more tile
  };
  // One tile in flight per wave and sixteen waves per CU (two tiles in flight do not fit the registers of that many).
  // Paged cache: the block-table lookup of the next tile is issued before the loads of this one, so that the wait for it
  // does not wait for them (memory operations complete in order).
  auto lookup = [&](int id) { return Rows::phys(page, b, lo + id); };
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
    auto offset = [&](int p) { return Rows::offset(page, p, stride_b, stride_n) * ES; };
    if constexpr (kKind == kKindFp8) Bt.fetch(Kbg, phys_now, lane, offset);
    else Bt.fetch(Kbg, phys_now, lane, offset, false);
  };
  Tile B0;
  int f0;
  if constexpr (kSplitLate) {
    request(B0, f0, 0);
    __builtin_amdgcn_sched_barrier(0);
    (void)query.operand(A, G, j);                        // (only fp16 has a range to report)
    for (int e0 = 0;;) {
      consume(B0, f0, e0);
      e0 += T;
      if (e0 >= cnt) break;
      request(B0, f0, e0);
    }
  } else {
    for (int e0 = 0; e0 < cnt; e0 += T) {
      request(B0, f0, e0);
      consume(B0, f0, e0);
    }
  }
  flush();
  leave(run);
}

// ----------------------------------------------------------------------------- launcher
int range_rows(const Shape& s, bool tables) { return range_rows_for((int64_t)s.B * s.Hkv, s.Lcap, s.G, tables); }

template <int G, bool kPaged, int kKind, bool kTables>
static constexpr auto range_kernel = &k_range_score<G, kPaged, kKind, kTables>;

hipError_t launch_range_score(const Shape& s, const float* q, const KvView& kv, const RangeSource& from,
                              const float* thr_state, float margin, float* tau_out, const int32_t* skip_if, float* score,
                              int32_t* slot_out, int64_t score_stride, int32_t* seg_count, int nseg, uint32_t* bitmap, int bitmap_words,
                              int range, int32_t* flags, hipStream_t st) {
  const int groups = s.B * s.Hkv, beside = groups % 8 == 0 ? 8 : 1;
  const int kind = kv.k_fp8 ? kKindFp8 : (kv.f16 ? kKindF16 : kKindBf16);
  const bool paged = kv.page.table != nullptr, tables = from.prev_topk == nullptr;
  hipError_t e = hipErrorInvalidValue;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(beside, (s.Lcap + range - 1) / range, groups / beside), dim3(kScoreThreads),
                       (size_t)range * 2, st, s, q, kv.k, kv.stride_b, kv.stride_h, kv.stride_n, kv.page, kv.seq_lens,
                       from, from.k, thr_state, margin, tau_out, skip_if, score, slot_out, score_stride, seg_count, nseg, bitmap, bitmap_words,
                       range, 0.08838834764831845f /* 1/sqrt(128) */, flags);
    e = hipGetLastError();
  };
  auto of_kind = [&](auto heads, auto pages, auto form) {
    constexpr int G = decltype(heads)::value;
    constexpr bool kPaged = decltype(pages)::value;
    if (kind != form.value) return;
    if (tables) launch(range_kernel<G, kPaged, decltype(form)::value, true>);
    else launch(range_kernel<G, kPaged, decltype(form)::value, false>);
  };
  auto of_pages = [&](auto heads, auto pages) {
    if (paged != pages.value) return;
    of_kind(heads, pages, std::integral_constant<int, kKindBf16>{});
    of_kind(heads, pages, std::integral_constant<int, kKindFp8>{});
    of_kind(heads, pages, std::integral_constant<int, kKindF16>{});
  };
  auto of_heads = [&](auto heads) {
    if (s.G != heads.value) return;
    of_pages(heads, std::false_type{});
    of_pages(heads, std::true_type{});
  };
  of_heads(std::integral_constant<int, 1>{});
  of_heads(std::integral_constant<int, 2>{});
  of_heads(std::integral_constant<int, 4>{});
  return e;
}

}  // namespace lfps
