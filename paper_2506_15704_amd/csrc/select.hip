// S3 — per query head, the k best of the scored rows (Alg. 1 line 8 / Sec. 1 Step 2).
//
// One workgroup (16 waves) per (b, h).
//
//  1. block min/max of the scores;
//  2. one LDS histogram of 2048 bins that are *linear in the score* between min and max.  (Bins
//     taken from the raw float bits would put a bell-shaped score distribution into a few dozen
//     bins and serialise the LDS atomics; linear bins spread it and leave only a handful of
//     scores in the bin that holds the k-th largest.)
//  3. the bin of the k-th largest score, by a suffix scan over the histogram;
//  4. the exact k-th largest inside that bin: its members go to a small LDS list and each is
//     ranked against the others; if the bin is too full for the list (degenerate inputs: all
//     scores equal, one huge outlier) an exact most-significant-digit radix descent over the
//     order-preserving 32-bit keys of the bin's members finds it instead;
//  5. ordered compaction (ballots and prefix counts; no atomics): every row above the k-th value plus as many rows
//     equal to it as still needed, lowest position first.  The output is ascending in position
//     and identical from run to run.
//
// Rows of more than 8192 scores whose scoring pass has left the largest score of every 16 are selected from the few blocks that
// hold the k best (select_blocks).  Other heads of up to kSelRegMax scores are read from memory once and stay in registers (select_regs.h); only when a row of
// 16384 to 32768 scores would keep more than the list of select_long holds (budgets of about 16000 and more, crowded
// bins) is it kept in LDS as a whole, and longer ones are streamed in each pass (L2).  32 heads x 32768 scores, k = 1024:
// 35 us with the row in LDS, 28 us with select_registers alone (32 elements a thread), 25 us this way (exact Top-k and attention of a 32K request: 57 -> 46 us).
// select_attend.hip applies the same to the short (score, position) lists that the filtered scoring pass leaves per
// head, and runs the attention over the selected rows in the same kernel.
#include "select_regs.h"

namespace lfps {

constexpr int kSelRegMax = 32 * kSelThreads;                // scores of a head that its workgroup's registers hold
constexpr int kSelListMax = kRegElems * kSelThreads;       // entries of select_long's list: 128 KB

__global__ __launch_bounds__(kSelThreads) void k_select(Shape s, const float* __restrict__ score,
                                                        int64_t score_stride, const int32_t* __restrict__ cand,
                                                        const int32_t* __restrict__ count_arr,
                                                        const int32_t* __restrict__ kk, int32_t* __restrict__ topk_idx,
                                                        float* __restrict__ topk_score, int list_cap,
                                                        int cache_elems, float* __restrict__ thr_state,
                                                        const int32_t* __restrict__ skip_if,
                                                        const int32_t* __restrict__ seq_lens,
                                                        const float* __restrict__ tops) {
  request_arguments<decltype(&k_select)>();
  constexpr int NT = kSelThreads;
  __shared__ SelectShared<NT> sm;
  extern __shared__ float dyn[];                    // select_long's list, or the scores of a whole row
  const int bh = blockIdx.x, b = bh / s.Hq, h = bh % s.Hq, g = h / s.G;
  const int tid = threadIdx.x;
  if (skip_if && skip_if[bh] != 0) return;          // bypassed head: its rows were written by the gate
  const bool gather = cand != nullptr;
  int c = gather ? count_arr[b * s.Hkv + g] : count_arr[b];
  const int c_max = gather ? s.cand_cap : s.Lcap;
  c = c < 0 ? 0 : (c > c_max ? c_max : c);
  int kb = kk[b];
  kb = kb < 0 ? 0 : (kb > s.kmax ? s.kmax : kb);
  const int ksel = kb < c ? kb : c;

  int32_t* oi = topk_idx + (int64_t)bh * s.kmax;
  float* os = topk_score ? topk_score + (int64_t)bh * s.kmax : nullptr;
  for (int i = ksel + tid; i < s.kmax; i += NT) {   // padding
    oi[i] = -1;
    if (os) os[i] = 0.f;
  }
  float* thr_out = thr_state ? thr_state + bh : nullptr;
  if (ksel == 0) {
    if (thr_out && tid == 0) *thr_out = -INFINITY;
    return;
  }

  const float* sc = score + (int64_t)bh * score_stride;
  const int32_t* cbg = gather ? cand + ((int64_t)b * s.Hkv + g) * s.cand_cap : nullptr;
  int n_valid = 0x7FFFFFFF;
  if (gather && seq_lens) {
    n_valid = seq_lens[b];
    n_valid = n_valid < 0 ? 0 : (n_valid > s.Lcap ? s.Lcap : n_valid);
  }
  auto put = [&](int rank, int e, float x) {
    const int p = cbg ? cbg[e] : e;
    const bool ok = (uint32_t)p < (uint32_t)n_valid;
    oi[rank] = ok ? p : -1;
    if (os) os[rank] = ok ? x : 0.f;
  };
  if (c <= 8 * NT) {                                // few scores: straight to the end
    for (int i = tid; i < 2 * NT; i += NT) sm.hist[i] = 0u;
    if (tid == 0) sm.list_n = 0u;
    __syncthreads();
    auto run = [&](auto elems) {
      constexpr int E = decltype(elems)::value;
      float v[E];
#pragma unroll
      for (int u = 0; u < E; ++u) v[u] = sc[u * NT + tid < c ? u * NT + tid : c - 1];
#pragma unroll
      for (int u = 0; u < E; ++u) v[u] = sanitize(v[u]);
      select_registers<NT, E>(sm, v, c, ksel, 0.f, true, thr_out,
                              [&](int rank, int u, float) { put(rank, u * NT + tid, v[u]); });
    };
    if (c <= 2 * NT) run(std::integral_constant<int, 2>{});
    else if (c <= 4 * NT) run(std::integral_constant<int, 4>{});
    else run(std::integral_constant<int, 8>{});
    return;
  }
  bool done = false;
  float2* list = reinterpret_cast<float2*>(dyn);
  static_assert(kTopsMinRows == 8 * NT && kTopsMaxRows == 16 * kRegElems * NT, "rows that select_blocks takes");
  if (tops && select_takes_tops(s, c, kb))
    done = select_blocks<NT>(sm, sc, tops + (int64_t)bh * (score_stride >> 4), c, ksel, list, list_cap, thr_out, put);
  if (done) return;
  if (c <= 16 * NT) done = select_long<NT, 16>(sm, sc, c, ksel, list, list_cap, thr_out, put);
  else if (c <= kSelRegMax) done = select_long<NT, 32>(sm, sc, c, ksel, list, list_cap, thr_out, put);
  if (done) return;
  __syncthreads();
  if (c <= cache_elems)
    select_body<true, NT>(sm, dyn, sc, c, ksel, cbg, oi, os, thr_out, n_valid);
  else
    select_stream(sm, sc, c, ksel, cbg, oi, os, thr_out, n_valid);
}

// LDS beside SelectShared: select_long's list, or the whole row where that would overflow.  (Rows of up to 8192 scores
// need neither.)
static void select_room(const Shape& s, bool gather, int* list_cap, int* cache_elems) {
  const int rows_max = gather ? s.cand_cap : s.Lcap;
  *cache_elems = rows_max <= 8 * kSelThreads ? 0 : (((rows_max < kCacheElems ? rows_max : kCacheElems) + 63) & ~63);
  *list_cap = rows_max <= 8 * kSelThreads ? 0 : kSelListMax;
}

// Are the largest scores of 16 rows each worth their writing by the scoring pass?  (They save the select most of its work, but
// where there are many heads the select's workgroups overlap and the writes do not.)  Exact Top-k of all rows, separate scores
// -> with tops: 1 x 32K 45.8 -> 36.0 us, 1 x 64K 95 -> 55, 4 x 30K 76 -> 68, 2 x 16K 35.1 -> 32.8, 6 x 16K 61.4 -> 59.7; but 8 x 16K
// (256 heads) 71.3 -> 72.5, 8 x 9000 49.3 -> 49.9, and rows of up to 8192 scores are selected without them.
bool select_wants_tops(const Shape& s) { return s.Lcap > 16384 || (s.Lcap > 8 * kSelThreads && s.B * s.Hq <= 192); }

// Called once per context at creation: the kernel needs more dynamic LDS than the default limit.
hipError_t configure_select(const Shape& s, int dtype, bool k_fp8, bool v_fp8) {
  hipError_t e = hipFuncSetAttribute((const void*)k_select, hipFuncAttributeMaxDynamicSharedMemorySize, kSelListMax * 8);
  if (e != hipSuccess) return e;
  return configure_select_attend(s, dtype, k_fp8, v_fp8);
}

hipError_t launch_select(const Shape& s, const float* score, int64_t score_stride, const int32_t* cand,
                         const int32_t* count, const int32_t* k, int32_t* topk_idx, float* topk_score,
                         float* thr_state, const int32_t* skip_if, const int32_t* seq_lens, hipStream_t st,
                         const float* tops) {
  int list_cap, cache_elems;
  select_room(s, cand != nullptr, &list_cap, &cache_elems);
  hipLaunchKernelGGL(k_select, dim3(s.B * s.Hq), dim3(kSelThreads), (size_t)(list_cap * 2 > cache_elems ? list_cap * 2 : cache_elems) * 4,
                     st, s, score, score_stride, cand, count, k, topk_idx, topk_score, list_cap, cache_elems, thr_state,
                     skip_if, seq_lens, tops);
  return hipGetLastError();
}

}  // namespace lfps
