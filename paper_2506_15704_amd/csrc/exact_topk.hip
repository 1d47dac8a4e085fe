// Exact Top-k baseline (Sec. 1 Steps 1-2 over all keys; the "exact Top-k" upper bound of Sec. 5), set-up of its
// fast form.  Writing a score for every row and selecting from that array costs a second and further passes over
// 4 bytes per row and head; instead the baseline takes the machinery of the chained steps:
//   1. a strided sample of each group's rows is scored (the gather kernel) and, per head, the sample score of a
//      rank chosen so that, with near certainty, between k rows and the select's list capacity reach it becomes a
//      threshold;
//   2. the filtered scoring kernel streams all rows once and keeps only those that reach the threshold;
//   3. the select picks the exact k best from the survivors; a head whose survivors are fewer than k (or too many
//      for the on-chip list) is rescored the plain way, so the result is always the exact Top-k.
#include "sample_plan.h"
#include "score_mfma.h"

namespace lfps {

// Step 1, the scores [B, Hq, ns] of the samples, and with them, by the first workgroup of every group, what the next steps need: its
// rows (x_cnt) and its place on the line of all rows (x_start, with the line's length behind), of every request the length of its
// samples and the rank (x_ns, x_rank).  grid (workgroups per group, B*Hkv).  (As a kernel before, which listed the sample rows, the
// set-up took 5.2 us and a boundary: exact Top-k of 8 x 64K with its attention 207.4 -> 203.4.)  One tile a wave, so what bounds it is
// the time to the first rows: with whole rows an instruction (StreamTile) and the query split behind the requests 16.8 -> 13.9 us, 42 MB of
// rows 6 KB apart, 204.9 -> 202.2 in all.  (Contiguous rows are better read the other way: exact Top-k of 1 x 32K 32.0 -> 32.4.)
template <int G, bool kPaged, int kKind>
__global__ __launch_bounds__(kScoreThreads) void k_sample_score(
    Shape s, const float* __restrict__ q, const void* __restrict__ K, int64_t stride_b, int64_t stride_h, int64_t stride_n, KvPage pg,
    const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ kk, int ns_max, int list_cap, int32_t* __restrict__ x_cnt,
    int64_t* __restrict__ x_start, int32_t* __restrict__ x_ns, int32_t* __restrict__ x_rank, float* __restrict__ score,
    int64_t score_stride, float scale, int32_t* __restrict__ flags) {
  request_arguments<decltype(&k_sample_score<G, kPaged, kKind>)>();
  const int bg = blockIdx.y, b = (int)((uint32_t)bg / (uint32_t)s.Hkv), g = bg - b * s.Hkv;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = lane & 15, kb = lane >> 4;
  auto len = [&](int bb) {
    const int n = seq_lens[bb];
    return n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  };
  const int n = len(b);
  const int k = kk[b] < 0 ? 0 : (kk[b] > s.kmax ? s.kmax : kk[b]);
  const SamplePlan plan = plan_sample(n, k, s.kmax > kSampleRanks ? s.kmax : kSampleRanks, ns_max, list_cap);
  if (blockIdx.x == 0 && wave == 0) {
    int64_t before = 0, all = 0;                            // rows of a head
    for (int bb = lane; bb < s.B; bb += 64) {
      const int64_t n_b = len(bb);
      before += bb < b ? n_b : 0;
      all += n_b;
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      before += __shfl_xor(before, d);
      all += __shfl_xor(all, d);
    }
    if (lane == 0) {
      x_cnt[bg] = n;
      x_start[bg] = before * s.Hkv + (int64_t)g * n;
      if (bg == 0) x_start[s.B * s.Hkv] = all * s.Hkv;
      if (g == 0) {
        x_ns[b] = plan.ns;
        x_rank[b] = plan.rank;
      }
    }
  }
  const int first = ((int)blockIdx.x * 4 + wave) * kRowsPerWaveIter;
  if (first >= plan.ns) return;
  using Op = typename KTile<kKind>::Operand;
  __shared__ u32x4 turn[kScoreThreads / 64][StreamTile<kKind>::kLdsChunks];
  Op A[4];
  QueryRows query;
  query.load(q, (int64_t)b * s.Hq + (int64_t)g * G, G, j, kb);
  const char* Kbg = static_cast<const char*>(K) + RowMap<kPaged>::base(b, g, stride_b, stride_h) * KTile<kKind>::kElemBytes;
  // row i of the sample: i n / ns, rounded down (the product is exact, and no quotient lies so near below a whole number that it would
  // be rounded up to it)
  score_slots_mfma<kPaged, kKind, false, true>(A, Kbg, pg, b, stride_b, stride_n, [&](int i) { return (int)((double)i * (double)n / (double)plan.ns); }, n,
                                  plan.ns, first, (int)gridDim.x * 4 * kRowsPerWaveIter,
                                  score + ((int64_t)b * s.Hq + (int64_t)g * G + kb) * score_stride, kb < G, scale, nullptr, turn[wave], &query,
                                  G, flags);
}

hipError_t launch_sample_score(const Shape& s, const float* q, const KvView& kv, const int32_t* k, int ns_max, int list_cap,
                               int32_t* x_cnt, int64_t* x_start, int32_t* x_ns, int32_t* x_rank, float* score, int64_t score_stride,
                               int32_t* flags, hipStream_t st) {
  const int most = ns_max < s.Lcap ? ns_max : s.Lcap, groups = s.B * s.Hkv;
  const int tiles = (most + 4 * kRowsPerWaveIter - 1) / (4 * kRowsPerWaveIter), want = (1024 + groups - 1) / groups;   // as launch_group_score
  const dim3 grid(tiles < want ? tiles : want, groups);
  const int kind = kv.k_fp8 ? kKindFp8 : (kv.f16 ? kKindF16 : kKindBf16);
  const bool paged = kv.page.table != nullptr;
  hipError_t e = hipErrorInvalidValue;
  auto launch = [&](auto heads, auto pages, auto form) {
    constexpr int G = decltype(heads)::value, kKind = decltype(form)::value;
    constexpr bool kPaged = decltype(pages)::value;
    if (s.G != G || paged != kPaged || kind != kKind) return;
    hipLaunchKernelGGL((k_sample_score<G, kPaged, kKind>), grid, dim3(kScoreThreads), 0, st, s, q, kv.k, kv.stride_b, kv.stride_h,
                       kv.stride_n, kv.page, kv.seq_lens, k, ns_max, list_cap, x_cnt, x_start, x_ns, x_rank, score, score_stride,
                       0.08838834764831845f /* 1/sqrt(128) */, flags);
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
