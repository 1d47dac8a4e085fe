// S3 + S4 in one kernel inside the chained steps: per query head the k best of its scored rows
// (Alg. 1 line 8 / Sec. 1 Step 2), then the attention output over exactly those rows (Eq. 1 / Sec. 1 Step 3).
// Both stages have one workgroup per (b, h); fused, the selected rows pass from one to the other in LDS, with their
// softmax numerators (the largest score, the softmax reference, is known from the select), heads that finish selecting
// early start gathering V rows while others still select, and a step has one kernel boundary less.
//
//   k_filter_select_attend   selects from the survivor lists that the filtered scoring pass leaves per head.
//                            A head whose survivors are fewer than k (or more than its registers hold) takes
//                            the unfiltered pass on the spot: its workgroup scores every candidate of the group
//                            for this head (the same MFMA arithmetic as the group scoring kernel, hence the same
//                            bits) into the head's score row and selects from that.  This is rare once a history
//                            exists (the threshold sits a margin below the previous k-th best score) and costs
//                            that workgroup the bytes of all candidate rows; in exchange a step has no conditional
//                            launches behind this kernel.
//   k_select_attend          selects from a head's full score row (all candidates): contexts without the filter.
//
// Both leave the k-th best score behind as the next step's threshold, but -inf (keep every candidate) for a head with
// fewer than ratio * k candidates, if they fill no more than half of the next step's list: there is little to filter then,
// and one head that the filter leaves short costs the step its unfiltered pass, 25 us.  The ratio is 2 for the memoryless
// form and 8 for the table form, whose candidate sets change in size by a half from one step to the next: table steps of
// 8 x 32K, k = 1024 of about 1300 candidates: 15 to 60 of 256 heads took the unfiltered pass, and this kernel 44 us instead
// of 19.  (Half of the list: with 5000 to 14000 candidates for lists of 4096 every head overflowed, 250 instead of 58 us.)
//
// For few heads both kernels are a chain of latencies: at 32 heads, k = 1024, the first one took 19.8 us, of which
// 1.8 us went into the piece counts, 6.3 into finding and fetching the survivors (twelve searches per thread, whatever
// their number, with 64-bit geometry), 4.4 into the select over LDS and 5.4 into the attention, which fetched the pairs
// back from global memory first.  Now the survivors go straight into registers (as many searches as a thread needs,
// 32-bit geometry) and stay there (select_regs.h), and the workgroup has as many threads as the number of heads leaves
// room for: 13 us (2.1 + 2.7 + 2.9 + 4.0); 512 heads, k = 2048: 45.8 -> 41 us, 1024 ragged heads: 52.7 -> 41 us.
#pragma once
#include "attend.h"
#include "range_geometry.h"
#include "score_mfma.h"
#include "select_regs.h"

#include <type_traits>

namespace lfps {

// Is the k-th best of c candidates a threshold worth remembering?  (keep: c < keep.ratio * k and c <= keep.most)
__device__ __forceinline__ bool filter_pays(int c, int ksel, const KeepAll& keep) {
  return c >= keep.ratio * ksel || c > keep.most;
}

// What a bypassed head remembers, by one thread: it has no k-th best score of this step.  -inf makes the first step in which
// it is not bypassed keep all candidates for it (the scoring pass keeps nothing for a bypassed head) and spares that step
// the unfiltered pass, which the score of an older step would often not.  But a head that had more candidates than half of
// the list in its last step would be sure to take that pass then: it keeps its score.  (Here, where nobody waits for it: in
// the gate's kernel the two loads cost each step 0.5 us.)
__device__ __forceinline__ void remember_bypassed(float* thr_state, const KeepAll& keep, int bh) {
  if (!(isfinite(thr_state[bh]) && keep.fits && keep.fits[bh] == 0)) thr_state[bh] = -INFINITY;
}

constexpr int kSelRowsMax = 16384;    // selected rows of a head that pass through LDS; more go through global memory

// Threads per head (16 waves per CU: the attention's loads in flight set the registers): as many as let every head's
// workgroup be resident at once, 1024 up to 256 heads, 512 up to 512, else 256; but the list holds kRegElems survivors per
// thread and has to hold four of the largest budget (1024 and 512 threads: two, or 7680).  Above 512 heads, steps whose
// heads all have enough survivors, 256 threads against 512: k = 128 46 against 52 us (608 heads) and 107 against 123
// (2048), k = 400 76 against 81 and 247 against 257, k = 1000 within 1 %; k = 1600 and 2048 equal, ragged budgets of
// 330 to 1311 2 % faster for four steps, but there a list of 4096 overflows, for every head at once, when the scores grow
// from one step to the next.  (The unfiltered pass of a head left short has half the waves: steps in which 2 % of the heads
// take it, k = 400, 193 against 175 us at 1024 heads.)
// Up to 64 heads with budgets of at most 512, whose candidates all fit the list of 512 threads: 512 (with four workgroups a head).  A
// head's uniform work is done by every wave on its own, and there are half as many; steps with 1024 -> 512, us: 1 x 3000, k = 48 16.5 ->
// 15.4, 1 x 16000, k = 256 17.3 -> 17.0, FP8 2 x 8000, k = 250 16.7 -> 16.4; k = 1024 27.0 -> 27.7, and with one workgroup a head within 1 %.
// With more candidates the unfiltered pass, of half the waves, costs what the other steps gain (four steps of 1 x 32K, k = 512, all heads
// of two of them short 356 -> 390), and a list half as long overflows where scores grow (2 x 120000, 34 rows around each of 512, scores
// times three 1280 -> 2620).
inline bool few_heads_short_lists(const Shape& s) { return s.B * s.Hq <= 64 && s.kmax <= 512 && s.cand_cap <= kRegElems * 512; }
inline int filter_select_threads(const Shape& s) {
  const int heads = s.B * s.Hq;
  if (few_heads_short_lists(s)) return 512;
  if (heads > 512 && kRegElems * 256 >= 4 * s.kmax) return 256;
  return heads <= 256 || kRegElems * 512 < 2 * s.kmax ? 1024 : 512;
}

// Attention over a head's rows as they stand in global memory (lists longer than kSelRowsMax).
template <typename T, int NW, bool kPaged>
static __device__ __noinline__ void attend_global(AttendShared& as, const T* V, int64_t stride_b, int64_t stride_h,
                                                  int64_t stride_n, const KvPage& page, int b, int g, int n, int kb,
                                                  const int32_t* oi, const float* os, float top, float* out_row) {
  attend_rows<T, NW, kPaged>(as, V, stride_b, stride_h, stride_n, page, b, g, n, kb, oi, os, true, top, out_row);
}

// Entries of weight 0 behind the ksel selected rows of a list, up to a multiple of 64 (and to `room`): the request's own row
// 0.  (Row 0 of a paged pool may belong to nobody, and 0 times what it holds need not be 0.)  Called by 64 threads or more.
template <bool kPaged>
__device__ __forceinline__ void pad_list(SelRow* list, const KvPage& page, int b, int ksel, int room) {
  if ((ksel & 63) == 0) return;                     // (uniform: the look-up is waited for by all)
  const int i = ksel + (int)threadIdx.x;
  if (i < ((ksel + 63) & ~63) && i < room) list[i] = SelRow{RowMap<kPaged>::phys(page, b, 0), 0.f};
}

// The rows a workgroup has just selected into global memory (oi, os; the caller's barrier has ordered the stores), as
// the attention's list.
template <int NT, bool kPaged>
__device__ __forceinline__ void list_from_global(SelRow* list, const KvPage& page, int b, int n, int ksel,
                                                 const int32_t* oi, const float* os, float top) {
  for (int i = threadIdx.x; i < ksel; i += NT) {
    const int r = oi[i];
    const bool ok = r >= 0 && r < n;
    list[i] = SelRow{RowMap<kPaged>::phys(page, b, ok ? r : 0), ok ? __expf(os[i] - top) : 0.f};
  }
}

// ----------------------------------------------------------------------------- from the survivor lists
// The filtered score kernel cuts the line of all groups' candidate slots into parts of S slots
// (S = *seg_rows_in), one per wave; my group starts at slot pg = group_start[b, g] of the line, and its piece
// `sgm` is what wave w_first + sgm took of it, w_first = pg / S: the group's slots [lo, hi).  The piece holds
// seg_count[bh, sgm] (score, row position) pairs at offset lo of the head's score / position rows, ascending in
// position within and across pieces.  Workgroup 0 leaves *line_total at zero for the next step.
// kRanges: the lists of the range kernel instead (range_geometry.h): piece counts are candidates << 16 | survivors, the
// group's candidate count is their sum (left in cand_count by the group's first head), the candidates are a bitmap.
// tau_in: per head, what the survivors have reached (thr_state is replaced while the kernel runs).
// The unfiltered pass needs the query, the K rows (format kKind) and the group's candidate list (cand; NULL when the
// candidates are all rows 0 .. count-1, the exact Top-k baseline's dense pass).
// kParts workgroups per head (attend_parts): all make the list, the first writes what a head leaves and alone takes the unfiltered pass, with all channels.
template <typename T, bool kPaged, int kKind, int NT, bool kRanges, int kParts>
__global__ __launch_bounds__(NT, 4) void k_filter_select_attend(
    Shape s, float* score, int32_t* slot, int64_t score_stride,
    const int32_t* __restrict__ seg_count, const int32_t* __restrict__ seg_rows_in, int nseg,
    const int32_t* __restrict__ cand, int32_t* __restrict__ cand_count, const int64_t* __restrict__ group_start,
    int64_t* __restrict__ line_total, int range_arg, const int32_t* __restrict__ parts_of, const uint32_t* __restrict__ bitmap, int bitmap_words,
    const int32_t* __restrict__ kk, int32_t* topk_idx, float* topk_score,
    float* __restrict__ thr_state, const float* __restrict__ tau_in, KeepAll keep, const int32_t* __restrict__ skip_if,
    int32_t* __restrict__ rescored,
    const float* __restrict__ q, const void* __restrict__ K, float scale, int32_t* __restrict__ flags,
    const T* __restrict__ V, int64_t stride_b, int64_t stride_h, int64_t stride_n, KvPage page,
    const int32_t* __restrict__ seq_lens, float* __restrict__ out) {
  constexpr int kWaves = NT / 64;
  constexpr int kPieces = 1024 / NT;               // pieces per thread: nseg <= 1024
  // Of paged rows, 1024 threads and lists on the line the registers are full, and the last lane's store of the wave's maximum costs
  // one more spilled (24 groups x 52567 bf16 rows: 16.8 us, through a scalar 16.3; where there is room the scalar is the slower way,
  // 64 groups x 32K contiguous rows, four steps, 238.7 -> 240.8).
  constexpr bool kScalarMax = kPaged && NT == 1024 && !kRanges;
  __shared__ SelectShared<NT> sm;
  __shared__ int seg_off[1024];
  __shared__ int wtot[kWaves], ctot[kWaves];
  __shared__ int btot[kWaves];                     // the bitmap scan's: ctot may still be read by a slower wave then
  extern __shared__ char dyn[];                    // the attention's partial sums, then the list of selected rows
  AttendShared& as = *reinterpret_cast<AttendShared*>(dyn);
  SelRow* list = reinterpret_cast<SelRow*>(dyn + sizeof(AttendShared));
  if (!kRanges && blockIdx.x == 0 && threadIdx.x == 0) *line_total = 0;   // the scoring pass that read it has finished
  request_arguments<decltype(&k_filter_select_attend<T, kPaged, kKind, NT, kRanges, kParts>)>();
  const HeadPlace at = place_of_block_for<kParts>(s.B, s.Hkv, s.G, blockIdx.x);     // the heads of a KV group on one XCD: they share V rows in its L2
  const int bh = at.bh, b = at.b, g = at.g, bg = at.bg, part = at.part;
  if (at.none) return;
  const bool writes = kParts == 1 || part == 0;
  const bool leads = writes && at.in_group == 0;     // leaves what the group's heads have in common
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool skipped = skip_if && skip_if[bh] != 0;  // bypassed head: its rows were written by the gate
  if (skipped && !(kRanges && leads)) {
    if (tid == 0 && writes) remember_bypassed(thr_state, keep, bh);
    return;
  }
  int raw[kPieces];                                  // piece counts of this head, masked once the geometry is known
#pragma unroll
  for (int u = 0; u < kPieces; ++u) {
    const int sgm = kPieces * tid + u;
    raw[u] = sgm < nseg ? seg_count[(int64_t)bh * nseg + sgm] : 0;
  }
  const float tau = tau_in[bh];                       // what the survivors have reached
  int c = kRanges ? 0 : cand_count[bg];
  const int strips = kRanges && parts_of ? 2 * parts_of[bg] : 0;
  int kb = kk[b];
  int n = seq_lens[b];
  int S = kRanges ? 64 : *seg_rows_in;                // chosen by the scoring pass of this step
  const int64_t pg = kRanges ? 0 : group_start[bg];
  c = c < 0 ? 0 : (c > s.cand_cap ? s.cand_cap : c);
  kb = kb < 0 ? 0 : (kb > s.kmax ? s.kmax : kb);
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  S = S < 64 ? 64 : S;
  // the group's slots relative to the part it starts in: piece sgm is [sgm * S - r0, (sgm + 1) * S - r0)
  const int r0 = (pg >> 32) == 0 ? (int)((uint32_t)pg % (uint32_t)S) : (int)(pg % S);
  const RangePieces geo(n, kRanges ? range_arg : 64, strips);
  int np = kRanges ? geo.count : (c > 0 ? (r0 + c - 1) / S + 1 : 0);         // pieces my group was cut into
  np = np > nseg ? nseg : np;
  auto piece_lo = [&](int sgm) { return kRanges ? geo.start(sgm) : (sgm > 0 ? sgm * S - r0 : 0); };

  // exclusive prefix of the piece counts (kPieces consecutive pieces per thread)
  for (int i = tid; i < 2 * NT; i += NT) sm.hist[i] = 0u;
  if (tid == 0) sm.list_n = 0u;
  int cntp[kPieces];
  int cnt = 0, cands = 0;
#pragma unroll
  for (int u = 0; u < kPieces; ++u) {
    const int sgm = kPieces * tid + u;
    cntp[u] = 0;
    if (sgm < np && kRanges) {
      const int room = geo.range >> 2;                             // rows the piece covers at most
      const int all = min(raw[u] >> 16 & 0xFFFF, room);
      cntp[u] = min(raw[u] & 0xFFFF, all);
      cands += all;
    } else if (sgm < np) {
      const int hi = (sgm + 1) * S - r0;
      const int room = (hi > c ? c : hi) - piece_lo(sgm);    // rows the piece covers
      cntp[u] = raw[u] < 0 ? 0 : (raw[u] > room ? room : raw[u]);
    }
    cnt += cntp[u];
  }
  const int inc = wave_inclusive_sum(cnt);
  if (lane == 63) wtot[wv] = inc;
  if (kRanges) {
    cands = wave_inclusive_sum(cands);
    if (lane == 63) ctot[wv] = cands;
  }
  __syncthreads();
  if (kRanges) {
    c += __builtin_amdgcn_readlane(wave_inclusive_sum(lane < kWaves ? ctot[lane] : 0), 63);
    if (tid == 0 && leads) cand_count[bg] = c;
    if (skipped) {
      if (tid == 0) remember_bypassed(thr_state, keep, bh);
      return;
    }
  }
  const int ksel = kb < c ? kb : c;
  const int of_wave = lane < kWaves ? wtot[lane] : 0, upto_wave = wave_inclusive_sum(of_wave);
  const int base = __builtin_amdgcn_readlane(upto_wave, wv) - __builtin_amdgcn_readlane(of_wave, wv);
  const int n_surv = __builtin_amdgcn_readlane(upto_wave, 63);
  {
    int off = base + inc - cnt;
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
      seg_off[kPieces * tid + u] = off;
      off += cntp[u];
    }
  }
  const bool unfiltered = n_surv < ksel || n_surv > kRegElems * NT;   // workgroup-uniform: the survivors cannot give the k best
  if (!writes && (unfiltered || ksel == 0)) return;
  if (unfiltered && tid == 0 && rescored) atomicAdd(rescored, 1);     // heads that took the unfiltered pass since the last poll
  int32_t* oi = topk_idx + (int64_t)bh * s.kmax;
  float* os = topk_score + (int64_t)bh * s.kmax;
  for (int i = ksel + tid; writes && i < s.kmax; i += NT) {   // padding
    oi[i] = -1;
    os[i] = 0.f;
  }
  pad_list<kPaged>(list, page, b, ksel, kSelRowsMax);
  if (ksel == 0) {
    if (tid == 0) thr_state[bh] = -INFINITY;
    if (out && tid < kD) out[(int64_t)bh * kD + tid] = 0.f;
    return;
  }
  float* thr_out = writes && filter_pays(c, ksel, keep) ? thr_state + bh : nullptr;
  if (tid == 0 && writes) {
    if (!thr_out) thr_state[bh] = -INFINITY;                // (nobody in this launch reads it: what the survivors reached is tau_in)
    if (keep.fits) keep.fits[bh] = c <= keep.most;
  }
  float* sc = score + (int64_t)bh * score_stride;
  int32_t* sl = slot + (int64_t)bh * score_stride;
  const int32_t* cbg = kRanges ? sl : (cand ? cand + (int64_t)bg * s.cand_cap : nullptr);
  if (unfiltered && kRanges) {                       // the group's candidates from the bitmap, ascending, over the survivors
    // A wave has consecutive words and expands eight at a time, so that its lanes store side by side.  (With a thread for consecutive words
    // of its own this took 25 us more for the 90000 candidates of a head, 575 us in all.)
    const uint32_t* bm = bitmap + (int64_t)bg * bitmap_words;
    const int W = (n + 31) >> 5, own = ((W + kWaves - 1) / kWaves + 7) & ~7;
    const int w0 = wv * own < W ? wv * own : W, w1 = w0 + own < W ? w0 + own : W;
    int mine = 0;
    for (int w = w0 + lane; w < w1; w += 64) mine += __popc(bm[w]);
    const int upto = wave_inclusive_sum(mine);
    if (lane == 63) btot[wv] = upto;
    __syncthreads();
    int at = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) at += w < wv ? btot[w] : 0;
    at = __builtin_amdgcn_readfirstlane(at);
    for (int w = w0; w < w1; w += 64) {
      const int word = w + lane < w1 ? (int)bm[w + lane] : 0;
      for (int i = 0; i < 64 && w + i < w1; i += 8) {
        const uint32_t four = (uint32_t)lane_value(word, (lane >> 3) + i, 0) >> (4 * (lane & 7)) & 15u;
        const int here = __popc(four), upto = wave_inclusive_sum(here), pos = ((w + i) << 5) + 4 * lane;
        int to = at + upto - here;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          if ((four >> p & 1u) && to < c) sl[to] = pos + p;
          to += four >> p & 1u;
        }
        at += __builtin_amdgcn_readlane(upto, 63);
      }
    }
    __syncthreads();
  }
  if (unfiltered) {
    // every candidate slot of the group, 64 per wave and visit, scored for the G heads; my head's lane group stores
    using Rows = RowMap<kPaged>;
    using Op = typename KTile<kKind>::Operand;
    Op A[4];
    report_q_range(load_query_operand(A, q, (int64_t)b * s.Hq + (int64_t)g * s.G, s.G, lane & 15, lane >> 4), flags);
    const char* Kbg = static_cast<const char*>(K) + Rows::base(b, g, stride_b, stride_h) * KTile<kKind>::kElemBytes;
    score_slots_mfma<kPaged, kKind>(A, Kbg, page, b, stride_b, stride_n, [&](int e) { return cbg ? cbg[e] : e; }, n, c, wv * kRowsPerWaveIter,
                                    kWaves * kRowsPerWaveIter, sc, (lane >> 4) == at.in_group, scale);
  }
  __syncthreads();                                  // seg_off, or the score row, is complete before anyone reads it
  const int n_el = unfiltered ? c : n_surv;
  if (n_el <= kRegElems * NT) {
    int topp = 1;
    while (topp < np) topp <<= 1;
    auto run = [&](auto elems) {
      constexpr int E = decltype(elems)::value;
      float v[E];
      int32_t pos[E], prow[E];
      if (unfiltered) {
#pragma unroll
        for (int u = 0; u < E; ++u) {
          const int e = u * NT + tid < n_el ? u * NT + tid : n_el - 1;
          v[u] = sc[e];
          pos[u] = cbg ? cbg[e] : e;
        }
      } else {
        // element e lies in the last piece with seg_off <= e (seg_off[0] = 0): E searches side by side, all loads
        // issued before the first is used
        int pc[E];
#pragma unroll
        for (int u = 0; u < E; ++u) pc[u] = 0;
        for (int half = topp >> 1; half >= 1; half >>= 1) {
#pragma unroll
          for (int u = 0; u < E; ++u) {
            const int mid = pc[u] + half;
            if (mid < np && seg_off[mid] <= u * NT + tid) pc[u] = mid;
          }
        }
#pragma unroll
        for (int u = 0; u < E; ++u) {
          const int e = u * NT + tid;
          const int src = e < n_el ? piece_lo(pc[u]) + (e - seg_off[pc[u]]) : piece_lo(pc[u]);
          v[u] = sc[src];
          pos[u] = sl[src];                              // the row position, written by the scoring pass
        }
      }
#pragma unroll
      for (int u = 0; u < E; ++u) {
        v[u] = sanitize(v[u]);
        const bool ok = pos[u] >= 0 && pos[u] < n;       // a bad entry of a caller's list is never a row
        if constexpr (E <= kRegElems / 2) prow[u] = RowMap<kPaged>::phys(page, b, ok ? pos[u] : 0);
        if (!ok) pos[u] = -1;
      }
      select_registers<NT, E, kScalarMax>(sm, v, n_el, ksel, tau, unfiltered || tau == -INFINITY, thr_out,
                                          [&](int rank, int u, float top) {
        const bool ok = pos[u] >= 0;
        if (writes) {
          oi[rank] = pos[u];
          os[rank] = ok ? v[u] : 0.f;
        }
        if constexpr (E > kRegElems / 2) prow[u] = RowMap<kPaged>::phys(page, b, ok ? pos[u] : 0);   // (registers)
        if (rank < kSelRowsMax) list[rank] = SelRow{prow[u], ok ? __expf(v[u] - top) : 0.f};
      });
    };
    if (n_el <= 2 * NT) run(std::integral_constant<int, 2>{});
    else if (n_el <= 4 * NT) run(std::integral_constant<int, 4>{});
    else if (n_el <= 8 * NT) run(std::integral_constant<int, 8>{});
    else run(std::integral_constant<int, kRegElems>{});
  } else {
    const float top = select_stream<NT>(sm, sc, c, ksel, cbg, oi, os, thr_out, n);
    __syncthreads();                                // this workgroup's stores of (position, score) before its loads of them
    if (ksel > kSelRowsMax) {
      if (out)
        attend_global<T, kWaves, kPaged>(as, V, stride_b, stride_h, stride_n, page, b, g, n, kb, oi, os, top,
                                         out + (int64_t)bh * kD);
      return;
    }
    list_from_global<NT, kPaged>(list, page, b, n, ksel, oi, os, top);
  }
  // ---- S4 over the rows just selected
  if (out == nullptr) return;                       // select only (the exact Top-k baseline)
  __syncthreads();
  const T* Vbg = V + RowMap<kPaged>::base(b, g, stride_b, stride_h);
  if (kParts > 1 && unfiltered)
    attend_list<T, kWaves, kPaged, 1>(as, Vbg, page, stride_b, stride_n, kb, ksel, list, out + (int64_t)bh * kD, 0);
  else
    attend_list<T, kWaves, kPaged, kParts>(as, Vbg, page, stride_b, stride_n, kb, ksel, list, out + (int64_t)bh * kD, part);
}

// ----------------------------------------------------------------------------- from the full score rows
// The k best of score[b, h, 0:c] (c = the group's candidate count), then the attention.  Rows that fit the workgroup's
// registers are selected there, up to kCacheElems in LDS, longer ones streamed.  kParts workgroups per head, as above: the first
// writes what a head leaves and alone takes rows that do not fit the registers, with all channels.
template <typename T, bool kPaged, int kParts>
__global__ __launch_bounds__(kSelThreads) void k_select_attend(
    Shape s, const float* __restrict__ score, int64_t score_stride, const int32_t* __restrict__ cand,
    const int32_t* __restrict__ cand_count, const int32_t* __restrict__ kk, int32_t* topk_idx, float* topk_score,
    int cache_elems, float* __restrict__ thr_state, KeepAll keep,
    const int32_t* __restrict__ skip_if, const T* __restrict__ V, int64_t stride_b, int64_t stride_h, int64_t stride_n,
    KvPage page, const int32_t* __restrict__ seq_lens, float* __restrict__ out) {
  constexpr int NT = kSelThreads;
  __shared__ SelectShared<NT> sm;
  __shared__ AttendShared as;
  extern __shared__ char dyn[];                     // the list of selected rows, or before it the scores of a long row
  SelRow* list = reinterpret_cast<SelRow*>(dyn);
  request_arguments<decltype(&k_select_attend<T, kPaged, kParts>)>();
  const HeadPlace at = place_of_block_for<kParts>(s.B, s.Hkv, s.G, blockIdx.x);
  const int bh = at.bh, b = at.b, g = at.g, part = at.part;
  if (at.none) return;
  const bool writes = kParts == 1 || part == 0;
  const int tid = threadIdx.x;
  if (skip_if && skip_if[bh] != 0) {                // bypassed head: its rows were written by the gate
    if (thr_state && tid == 0 && writes) remember_bypassed(thr_state, keep, bh);
    return;
  }
  int c = cand_count[at.bg];
  c = c < 0 ? 0 : (c > s.cand_cap ? s.cand_cap : c);
  int kb = kk[b];
  kb = kb < 0 ? 0 : (kb > s.kmax ? s.kmax : kb);
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const int ksel = kb < c ? kb : c;
  const bool in_registers = c <= kRegElems * NT;
  if (!writes && (!in_registers || ksel == 0)) return;
  int32_t* oi = topk_idx + (int64_t)bh * s.kmax;
  float* os = topk_score + (int64_t)bh * s.kmax;
  for (int i = ksel + tid; writes && i < s.kmax; i += NT) {   // padding
    oi[i] = -1;
    os[i] = 0.f;
  }
  float* thr_out = thr_state && writes ? thr_state + bh : nullptr;
  if (ksel == 0) {
    if (thr_out && tid == 0) *thr_out = -INFINITY;
    if (tid < kD) out[(int64_t)bh * kD + tid] = 0.f;
    return;
  }
  if constexpr (!std::is_same<T, float>::value) {   // (no filter for fp32 caches)
    if (keep.fits && tid == 0 && writes) keep.fits[bh] = c <= keep.most;
  }
  if (thr_out && !filter_pays(c, ksel, keep)) {
    if (tid == 0) *thr_out = -INFINITY;
    thr_out = nullptr;
  }
  const float* sc = score + (int64_t)bh * score_stride;
  const int32_t* cbg = cand + (int64_t)at.bg * s.cand_cap;
  if (in_registers) {
    for (int i = tid; i < 2 * NT; i += NT) sm.hist[i] = 0u;
    if (tid == 0) sm.list_n = 0u;
    pad_list<kPaged>(list, page, b, ksel, kSelRowsMax);
    __syncthreads();
    auto run = [&](auto elems) {
      constexpr int E = decltype(elems)::value;
      float v[E];
      int32_t pos[E], prow[E];
#pragma unroll
      for (int u = 0; u < E; ++u) {
        const int e = u * NT + tid < c ? u * NT + tid : c - 1;
        v[u] = sc[e];
        pos[u] = cbg[e];
      }
#pragma unroll
      for (int u = 0; u < E; ++u) {
        v[u] = sanitize(v[u]);
        const bool ok = pos[u] >= 0 && pos[u] < n;
        if constexpr (E <= kRegElems / 2) prow[u] = RowMap<kPaged>::phys(page, b, ok ? pos[u] : 0);
        if (!ok) pos[u] = -1;
      }
      select_registers<NT, E>(sm, v, c, ksel, 0.f, true, thr_out, [&](int rank, int u, float top) {
        const bool ok = pos[u] >= 0;
        if (writes) {
          oi[rank] = pos[u];
          os[rank] = ok ? v[u] : 0.f;
        }
        if constexpr (E > kRegElems / 2) prow[u] = RowMap<kPaged>::phys(page, b, ok ? pos[u] : 0);
        list[rank] = SelRow{prow[u], ok ? __expf(v[u] - top) : 0.f};
      });
    };
    if (c <= 2 * NT) run(std::integral_constant<int, 2>{});
    else if (c <= 4 * NT) run(std::integral_constant<int, 4>{});
    else if (c <= 8 * NT) run(std::integral_constant<int, 8>{});
    else run(std::integral_constant<int, kRegElems>{});
  } else {
    float top;
    if (c <= cache_elems)
      select_body<true, NT>(sm, reinterpret_cast<float*>(dyn), sc, c, ksel, cbg, oi, os, thr_out, n, &top);
    else
      top = select_stream(sm, sc, c, ksel, cbg, oi, os, thr_out, n);
    __syncthreads();                                // this workgroup's stores of (position, score) before its loads of them
    if (ksel > kSelRowsMax) {
      attend_global<T, NT / 64, kPaged>(as, V, stride_b, stride_h, stride_n, page, b, g, n, kb, oi, os, top,
                                        out + (int64_t)bh * kD);
      return;
    }
    pad_list<kPaged>(list, page, b, ksel, kSelRowsMax);
    list_from_global<NT, kPaged>(list, page, b, n, ksel, oi, os, top);
  }
  __syncthreads();
  const T* Vbg = V + RowMap<kPaged>::base(b, g, stride_b, stride_h);
  if (kParts > 1 && !in_registers)
    attend_list<T, NT / 64, kPaged, 1>(as, Vbg, page, stride_b, stride_n, kb, ksel, list, out + (int64_t)bh * kD, 0);
  else
    attend_list<T, NT / 64, kPaged, kParts>(as, Vbg, page, stride_b, stride_n, kb, ksel, list, out + (int64_t)bh * kD, part);
}

// ----------------------------------------------------------------------------- launchers
// LDS of the list of selected rows.
inline int sel_list_bytes(const Shape& s) {
  const int rows = s.kmax < kSelRowsMax ? s.kmax : kSelRowsMax;
  return ((rows + 63) & ~63) * (int)sizeof(SelRow);
}
// k_select_attend keeps long score rows in LDS as well.
inline int select_attend_cache(const Shape& s) {
  const int ce = ((s.cand_cap < kCacheElems ? s.cand_cap : kCacheElems) + 63) & ~63;
  return ce > kRegElems * kSelThreads ? ce : 0;
}

inline int most_kept(const Shape& s) { return few_heads_short_lists(s) ? filter_list_cap(s) : filter_list_cap(s) / 2; }

// What the launches below are made from.
struct FilterSelectArgs {
  Shape s;
  float* score;
  int32_t* slot;
  int64_t score_stride;
  const int32_t* seg_count;
  const int32_t* seg_rows;
  int nseg;
  const int32_t* cand;
  int32_t* cand_count;
  const int64_t* group_start;
  int64_t* line_total;
  int range;
  const int32_t* parts_of;
  const uint32_t* bitmap;
  int bitmap_words;
  const int32_t* k;
  int32_t* topk_idx;
  float* topk_score;
  float* thr_state;
  const float* tau;
  KeepAll keep;
  const int32_t* skip_if;
  int32_t* rescored;
  const float* q;
  int32_t* flags;
  const KvView* kv;
  float* out;
};
struct SelectArgs {
  Shape s;
  const float* score;
  int64_t score_stride;
  const int32_t* cand;
  const int32_t* cand_count;
  const int32_t* k;
  int32_t* topk_idx;
  float* topk_score;
  float* thr_state;
  KeepAll keep;
  const int32_t* skip_if;
  const KvView* kv;
  float* out;
};

// The instantiations for values of type T: paged or not, the threads per head, the form of the lists, the workgroups per head.
// use(kernel, paged, threads, ranges, parts) for each.  (Files of their own, one per type of values: they take long to compile.)
template <typename T, int kKind, typename Use>
void each_filter_select(Use use) {
  auto of = [&](auto paged, auto ranges) {
    constexpr bool kPaged = decltype(paged)::value, kRanges = decltype(ranges)::value;
    use(&k_filter_select_attend<T, kPaged, kKind, 256, kRanges, 1>, kPaged, 256, kRanges, 1);
    use(&k_filter_select_attend<T, kPaged, kKind, 512, kRanges, 1>, kPaged, 512, kRanges, 1);
    use(&k_filter_select_attend<T, kPaged, kKind, 1024, kRanges, 1>, kPaged, 1024, kRanges, 1);
    use(&k_filter_select_attend<T, kPaged, kKind, 512, kRanges, 4>, kPaged, 512, kRanges, 4);
    use(&k_filter_select_attend<T, kPaged, kKind, 1024, kRanges, 4>, kPaged, 1024, kRanges, 4);
  };
  of(std::false_type{}, std::false_type{});
  of(std::false_type{}, std::true_type{});
  of(std::true_type{}, std::false_type{});
  of(std::true_type{}, std::true_type{});
}
template <typename T, typename Use>
void each_select(Use use) {
  use(&k_select_attend<T, false, 1>, false, 1);
  use(&k_select_attend<T, false, 4>, false, 4);
  use(&k_select_attend<T, true, 1>, true, 1);
  use(&k_select_attend<T, true, 4>, true, 4);
}

// The kernels that the steps of a context can launch may need more dynamic LDS than the default limit.  The limit belongs to the
// kernel and not to the context, so it is set to the most that any context asks for.
inline hipError_t raise_lds(const void* kernel, int bytes) {
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}
template <typename T, int kKind>
hipError_t configure_filter_select(const Shape& s) {
  Shape dense = s;                                         // (the exact Top-k, with all rows for candidates)
  dense.cand_cap = s.Lcap;
  hipError_t e = hipSuccess;
  each_filter_select<T, kKind>([&](auto kernel, bool, int threads, bool, int) {
    if (e == hipSuccess && (threads == filter_select_threads(s) || threads == filter_select_threads(dense)))
      e = raise_lds((const void*)kernel, (int)sizeof(AttendShared) + kSelRowsMax * (int)sizeof(SelRow));
  });
  return e;
}
template <typename T>
hipError_t configure_select_only(const Shape& s) {
  hipError_t e = hipSuccess;
  each_select<T>([&](auto kernel, bool, int) {
    if (e == hipSuccess) e = raise_lds((const void*)kernel, kCacheElems * 4);
  });
  return e;
}

template <typename T, int kKind>
hipError_t launch_filter_select(const FilterSelectArgs& a, hipStream_t st) {
  const int nt = filter_select_threads(a.s), parts = a.out ? attend_parts(a.s, *a.kv) : 1;
  const bool paged = a.kv->page.table != nullptr;
  const KvView& kv = *a.kv;
  KeepAll keep = a.keep;
  keep.most = most_kept(a.s);
  bool launched = false;
  each_filter_select<T, kKind>([&](auto kernel, bool of_pages, int threads, bool ranges, int of_head) {
    if (paged != of_pages || nt != threads || (a.range > 0) != ranges || parts != of_head) return;
    hipLaunchKernelGGL(kernel, dim3(attend_blocks(a.s, parts)), dim3(nt), (size_t)(sizeof(AttendShared) + sel_list_bytes(a.s)), st, a.s,
                       a.score, a.slot, a.score_stride, a.seg_count, a.seg_rows, a.nseg, a.cand, a.cand_count, a.group_start,
                       a.line_total, a.range, a.parts_of, a.bitmap, a.bitmap_words, a.k, a.topk_idx, a.topk_score, a.thr_state, a.tau, keep,
                       a.skip_if, a.rescored, a.q, kv.k, 0.08838834764831845f /* 1/sqrt(128) */, a.flags, (const T*)kv.v, kv.stride_b,
                       kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, a.out);
    launched = true;
  });
  return launched ? hipGetLastError() : hipErrorInvalidValue;
}
template <typename T>
hipError_t launch_select_only(const SelectArgs& a, hipStream_t st) {
  const int cache = select_attend_cache(a.s), parts = attend_parts(a.s, *a.kv);
  const int lds = cache * 4 > sel_list_bytes(a.s) ? cache * 4 : sel_list_bytes(a.s);
  const bool paged = a.kv->page.table != nullptr;
  const KvView& kv = *a.kv;
  KeepAll keep = a.keep;
  keep.most = most_kept(a.s);
  each_select<T>([&](auto kernel, bool of_pages, int of_head) {
    if (paged != of_pages || parts != of_head) return;
    hipLaunchKernelGGL(kernel, dim3(attend_blocks(a.s, parts)), dim3(kSelThreads), (size_t)lds, st, a.s, a.score, a.score_stride, a.cand,
                       a.cand_count, a.k, a.topk_idx, a.topk_score, cache, a.thr_state, keep, a.skip_if, (const T*)kv.v, kv.stride_b,
                       kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, a.out);
  });
  return hipGetLastError();
}

}  // namespace lfps
