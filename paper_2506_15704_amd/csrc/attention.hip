// S4 — sparse attention over the selected rows (Eq. 1), and the full-attention baseline
// (Sec. 1 with idx = every row; the "full attention" upper bound of Sec. 5).
//
// Sparse: the scores of the selected rows are already known (from S3, or recomputed by the
// per-head score kernel), so the softmax maximum is known before any V row is read and the
// partial sums of the waves merge by plain addition.  One workgroup of 4, 8 or 16 waves per
// (b, h): wave w gathers its share of the head's rows, 16 lanes per V row, 16-byte loads, sixteen
// independent row loads in flight per wave; the partial sums meet in LDS and the output row is
// written once (no partials in global memory, no second kernel).
//
// Full: split-K over contiguous row ranges with the G heads of a group sharing every K and V row; a wave keeps the running
// (max, sum, acc) of its heads, without grouping a lane group of 16 that of its rows, merged with the online-softmax rule.
#include "attend.h"

namespace lfps {

constexpr int kAttnThreads = 256;       // full attention

// grid B*Hq * kParts, kSparseWaves waves per workgroup
template <typename T, int kSparseWaves, bool kPaged, int kParts>
__global__ __launch_bounds__(kSparseWaves * 64) void k_sparse_attn(Shape s, const T* __restrict__ V, int64_t stride_b,
                                                                int64_t stride_h, int64_t stride_n, KvPage pg,
                                                                const int32_t* __restrict__ seq_lens,
                                                                const int32_t* __restrict__ idx,
                                                                const float* __restrict__ idx_score,
                                                                const int32_t* __restrict__ kk,
                                                                float* __restrict__ out,
                                                                const int32_t* __restrict__ skip_if) {
  __shared__ AttendShared sm;
  request_arguments<decltype(&k_sparse_attn<T, kSparseWaves, kPaged, kParts>)>();
  const HeadPlace at = place_of_block_for<kParts>(s.B, s.Hkv, s.G, blockIdx.x);
  const int bh = at.bh, b = at.b, g = at.g;
  if (at.none) return;
  if (skip_if && skip_if[bh] != 0) return;            // bypassed head: the gate wrote its output row
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  int kb = kk[b];
  kb = kb < 0 ? 0 : (kb > s.kmax ? s.kmax : kb);
  attend_rows<T, kSparseWaves, kPaged, kParts>(sm, V, stride_b, stride_h, stride_n, pg, b, g, n, kb,
                                               idx + (int64_t)bh * s.kmax, idx_score + (int64_t)bh * s.kmax, false, 0.f,
                                               out + (int64_t)bh * kD, at.part);
}

template <typename T>
static hipError_t launch_sparse_t(const Shape& s, const KvView& kv, const int32_t* idx, const float* idx_score,
                                  const int32_t* k, float* out, const int32_t* skip_if, hipStream_t st) {
  // as many waves per head as keep every head's workgroup resident at once (256 CUs x 32 waves)
  const int heads = s.B * s.Hq;
  const T* V = (const T*)kv.v;
#define LFPS_LAUNCH_SPARSE_P(NW, PAGED, PARTS)                                                                           \
  hipLaunchKernelGGL((k_sparse_attn<T, NW, PAGED, PARTS>), dim3(attend_blocks(s, PARTS)), dim3(NW * 64), 0, st, s, V, kv.stride_b, \
                     kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, idx, idx_score, k, out, skip_if)
#define LFPS_LAUNCH_SPARSE(NW, PARTS)          \
  if (kv.page.table) {                         \
    LFPS_LAUNCH_SPARSE_P(NW, true, PARTS);     \
  } else {                                     \
    LFPS_LAUNCH_SPARSE_P(NW, false, PARTS);    \
  }
  if (attend_parts(s, kv) == 4) {
    LFPS_LAUNCH_SPARSE(16, 4)
  } else if (heads * 16 <= 4096) {
    LFPS_LAUNCH_SPARSE(16, 1)
  } else if (heads * 8 <= 4096) {
    LFPS_LAUNCH_SPARSE(8, 1)
  } else {
    LFPS_LAUNCH_SPARSE(4, 1)
  }
#undef LFPS_LAUNCH_SPARSE
#undef LFPS_LAUNCH_SPARSE_P
  return hipGetLastError();
}

hipError_t launch_sparse_attn(const Shape& s, int dtype, const KvView& kv, const int32_t* idx, const float* idx_score,
                              const int32_t* k, float* out, const int32_t* skip_if, hipStream_t st) {
  if (dtype == LFPS_BF16 && kv.v_fp8) return launch_sparse_t<uint8_t>(s, kv, idx, idx_score, k, out, skip_if, st);
  if (dtype == LFPS_F16) return launch_sparse_t<_Float16>(s, kv, idx, idx_score, k, out, skip_if, st);
  return dtype == LFPS_BF16 ? launch_sparse_t<uint16_t>(s, kv, idx, idx_score, k, out, skip_if, st)
                            : launch_sparse_t<float>(s, kv, idx, idx_score, k, out, skip_if, st);
}

// ============================================================================ full attention
int full_attn_splits(const Shape& s) {
  int ns = (2048 + s.B * s.Hkv - 1) / (s.B * s.Hkv);
  int by_len = (s.Lcap + 255) / 256;       // at least 256 rows per split
  if (ns > by_len) ns = by_len;
  if (ns > kMaxSplits) ns = kMaxSplits;
  return ns < 1 ? 1 : ns;
}

__device__ __forceinline__ int rows_per_split(int n, int n_split) { return (((n + n_split - 1) / n_split) + 15) & ~15; }

// x[u] = the elements at at(u), past the caches or not.  (A choice at run time between the two forms of one load is merged by the
// compiler, into the ordinary one: the kernels hold their loops twice.)
template <bool kOnce, typename Raw, int U, typename At>
__device__ __forceinline__ void load_rows(Raw (&x)[U], At at) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if constexpr (kOnce) x[u].load_once(at(u));
    else x[u].load(at(u));
  }
}

// The weight of a partial result whose largest score lies x <= 0 from the largest of all.  Without grouping the scores are held as
// powers of two (k_full_attn_single).
template <int G>
__device__ __forceinline__ float part_weight(float x) { return G == 1 ? __builtin_amdgcn_exp2f(x) : exp_below<false>(x); }

// The four waves of a workgroup (a wave without rows: m = -inf, weight 0) -> po [G, D+2]: acc[D], m, l.  All threads call, after a
// barrier.
template <int G>
__device__ __forceinline__ void merge_waves(const float (&red_acc)[4][G][kD], const float (&red_m)[4][G],
                                            const float (&red_l)[4][G], float* __restrict__ po) {
  for (int e = threadIdx.x; e < G * kD; e += kAttnThreads) {
    const int h = e / kD, c = e % kD;
    const float mx = fmaxf(fmaxf(red_m[0][h], red_m[1][h]), fmaxf(red_m[2][h], red_m[3][h]));
    float a = 0.f, ls = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = (red_m[w][h] == -INFINITY) ? 0.f : part_weight<G>(red_m[w][h] - mx);
      a = fmaf(red_acc[w][h][c], f, a);
      ls = fmaf(red_l[w][h], f, ls);
    }
    po[h * (kD + 2) + c] = a;
    if (c == 0) {
      po[h * (kD + 2) + kD] = mx;
      po[h * (kD + 2) + kD + 1] = ls;
    }
  }
}

// The sums over the 16 lanes of a row of lanes of a[0 .. G-1], G = 2 or 4: lane j receives that of a[j % G].  (A butterfly
// over lane distances 1, 2, 4, 8 in which the first log2 G steps also share the G sums out: 11 instructions instead of 16.)
template <int G>
__device__ __forceinline__ float row16_shared_sums(float (&a)[G], int j) {
#define LFPS_DPP(v, ctrl) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, false))
  const bool odd = j & 1;
  float x, y[G / 2];
#pragma unroll
  for (int h = 0; h < G / 2; ++h) {
    const float keep = odd ? a[2 * h + 1] : a[2 * h], give = odd ? a[2 * h] : a[2 * h + 1];
    y[h] = keep + LFPS_DPP(give, 0xB1);                      // quad_perm 1 0 3 2
  }
  if constexpr (G == 2) {
    x = y[0];
    x += LFPS_DPP(x, 0x4E);                                  // quad_perm 2 3 0 1
  } else {
    const bool upper = j & 2;
    const float keep = upper ? y[1] : y[0], give = upper ? y[0] : y[1];
    x = keep + LFPS_DPP(give, 0x4E);
  }
  // (lanes j and j ^ 4, then j ^ 8, by rotation: every lane of a quad holds another sum)
  x += row16_rotate<4>(x);                                   // with the next one, the pairs' sums agree
  x += row16_rotate<8>(x);
  return x;
#undef LFPS_DPP
}

// G = 2 or 4.  grid (n_split, B*Hkv); part [B*Hkv, n_split, G, D+2]: acc[D], m, l
//
// A wave takes U groups of four rows at a time, 16 lanes a row, 8 channels a lane, for K and for V.  The G sums of a row are
// shared out over its lanes, so that a lane makes the softmax step for one head and its own rows only, once per tile; the
// weights reach the lanes that hold the values through LDS.  The rows of K and of V are in flight in turn, those of one while
// the other is used.  Bound by the bytes of K and V in 16 bits (64 groups x 32K rows, 1.07 GB: 168.5 us with the merge, 199 with an
// earlier form), by the multiply-adds in FP8 (the same rows: 112 us, 233): when every lane made the step for all heads and each of
// its rows, a row cost the same whatever it took to fetch.  U = 16 for FP8 leaves two waves per SIMD: 13 us slower.
// Rows of a contiguous cache are counted, not looked up across lanes, which made every load wait for LDS: bf16 172.5 -> 168.5 us, FP8
// 114 -> 112, 8 x 16384 in FP8 57.2 -> 56.9, 16 x 8480 60.0 -> 59.3.
// (The dot products on the matrix units were as fast, 169 to 180 us, but 1.3 times as far from 64 bits where a few rows carry
// the weight: large scores are sums of like-signed products there.)
// kMayOnce: rows past the caches where the rows that the requests hold outgrow the memory-side cache (kKeptStreamBytes; 8 x 32K rows 195 against
// 207 us with the kernel as it was); fewer are found there by the next call, whatever the context has room for (8 x 8192 of
// 131072 rows in bf16 52.9 -> 48.8 us, 8 x 16384 in FP8 62.3 -> 57.3, against that capacity deciding).
template <typename TK, typename T, int G, bool kPaged, bool kMayOnce>
__global__ __launch_bounds__(kAttnThreads) void k_full_attn(Shape s, const float* __restrict__ q,
                                                            const TK* __restrict__ K, const T* __restrict__ V,
                                                            int64_t stride_b, int64_t stride_h, int64_t stride_n,
                                                            KvPage pg, const int32_t* __restrict__ seq_lens,
                                                            float* __restrict__ part, int n_split, float scale) {
  constexpr int U = sizeof(TK) == 4 ? 4 : 8, kRows = 4 * U;
  constexpr int kShare = 16 / G;                            // lanes of a row that hold the same head's sum
  constexpr int NV = U > kShare ? U / kShare : 1;           // (row, head) pairs of a lane
  __shared__ float red_acc[4][G][kD];
  __shared__ float weight[4][kRows][G];
  __shared__ float red_m[4][G], red_l[4][G];
  const int bg = blockIdx.y, b = bg / s.Hkv, g = bg % s.Hkv, split = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, rs = lane >> 4;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const int rps = rows_per_split(n, n_split);
  const int r_begin = split * rps;
  const int r_end = (r_begin + rps < n) ? r_begin + rps : n;
  if (r_begin >= n) return;
  const bool once_here = kMayOnce && outgrow_cache(s, held_rows(s, seq_lens), kD * (int)(sizeof(TK) + sizeof(T)), kKeptStreamBytes);

  float qr[G][8];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float* qh = q + ((int64_t)b * s.Hq + (int64_t)g * G + h) * kD + 8 * j;
#pragma unroll
    for (int c = 0; c < 8; ++c) qr[h][c] = qh[c] * scale;
  }
  using Rows = RowMap<kPaged>;
  const TK* Kbg = K + Rows::base(b, g, stride_b, stride_h) + 8 * j;
  const T* Vbg = V + Rows::base(b, g, stride_b, stride_h) + 8 * j;
  // Rows past the end are read from the last row and weigh nothing, so no load sits behind a branch.
  auto clamped = [&](int r) { return r < r_end ? r : r_end - 1; };
  // the tile at r0: paged, its row r0 + lane as a physical row; else its first row
  auto rows_of = [&](int r0) { return kPaged ? Rows::phys(pg, b, clamped(r0 + lane)) : r0; };
  auto row_value = [&](int x, int u) {                      // of row 4 u + rs
    return kPaged ? __builtin_amdgcn_ds_bpermute(4 * rs + 16 * u, x) : clamped(x + 4 * u + rs);
  };
  Raw8<TK> kt[U];                                           // kt[u], vt[u]: my channels of row 4 u + rs
  Raw8<T> vt[U];
  auto fetch_k = [&](auto once, int phys) {
    load_rows<decltype(once)::value>(kt, [&](int u) { return Kbg + Rows::offset(pg, row_value(phys, u), stride_b, stride_n); });
  };
  auto fetch_v = [&](auto once, int phys) {
    load_rows<decltype(once)::value>(vt, [&](int u) { return Vbg + Rows::offset(pg, row_value(phys, u), stride_b, stride_n); });
  };
  // my pairs: head j % G and the rows 4 u + rs with u = t * kShare + j / G
  const int my_u = j / G;
  const bool mine = my_u < U;
  float m = -INFINITY, l = 0.f;                             // of head j % G: largest score so far; the sum over my rows
  float acc[G][8];
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[h][c] = 0.f;

  constexpr int kStep = 4 * kRows;                          // wave w takes tiles w, w + 4, ...
  auto walk = [&](auto once) {
  int r0 = r_begin + kRows * wave;
  int phys = rows_of(r0), phys_next = rows_of(r0 + kStep);
  fetch_k(once, phys);
  fetch_v(once, phys);
  for (; r0 < r_end; r0 += kStep) {
    float v[NV];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float x[8], a[G];
      kt[u].get(x);
#pragma unroll
      for (int h = 0; h < G; ++h) {
        a[h] = qr[h][0] * x[0];
#pragma unroll
        for (int c = 1; c < 8; ++c) a[h] = fmaf(qr[h][c], x[c], a[h]);
      }
      const float sum = row16_shared_sums<G>(a, j);
      v[u / kShare] = u % kShare == 0 || my_u == u % kShare ? sum : v[u / kShare];
      if (u % 2) __builtin_amdgcn_sched_barrier(0);         // (registers: two rows' elements at a time as fp32)
    }
    phys = phys_next;
    phys_next = rows_of(r0 + 2 * kStep);
    if constexpr (kPaged) __builtin_amdgcn_sched_barrier(0);      // the look-up before the rows: its wait must not include them
    fetch_k(once, phys);
    // one online-softmax step
    bool ok[NV];
    float mx = m;
#pragma unroll
    for (int t = 0; t < NV; ++t) {
      ok[t] = mine && r0 + 4 * (t * kShare + my_u) + rs < r_end;
      mx = ok[t] ? fmaxf(mx, v[t]) : mx;
    }
    mx = fmaxf(mx, row16_rotate<8>(mx));
    mx = fmaxf(mx, row16_rotate<4>(mx));
    if constexpr (G == 2) mx = fmaxf(mx, row16_rotate<2>(mx));
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float alpha = mx == -INFINITY ? 1.f : exp_below<false>(m - mx);      // (0 on the first tile)
    l *= alpha;
    m = mx;
    wave_lds_order();                                                // (the weights of the tile before have been read)
#pragma unroll
    for (int t = 0; t < NV; ++t) {
      const float e = exp_below<false>(v[t] - mx);
      const float p = ok[t] && v[t] != -INFINITY ? e : 0.f;
      l += p;
      if (mine) weight[wave][4 * (t * kShare + my_u) + rs][j % G] = p;
    }
    wave_lds_order();
    if (__ballot(alpha != 1.f)) {
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(alpha), h));
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[h][c] *= a;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float x[8], p[G];
      vt[u].get(x);
#pragma unroll
      for (int h = 0; h < G; ++h) p[h] = weight[wave][4 * u + rs][h];
#pragma unroll
      for (int h = 0; h < G; ++h)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[h][c] = fmaf(p[h], x[c], acc[h][c]);
      if (u % 2) __builtin_amdgcn_sched_barrier(0);
    }
    fetch_v(once, phys);
  }
  };
  if (once_here) walk(std::true_type{});
  else walk(std::false_type{});

  // the lanes of the wave, then the four waves (a wave without rows: m = -inf, weight 0)
#pragma unroll
  for (int d = G; d < 64; d <<= 1) l += __shfl_xor(l, d);
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      acc[h][c] += __shfl_xor(acc[h][c], 16);
      acc[h][c] += __shfl_xor(acc[h][c], 32);
    }
  if (rs == 0) {
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int c = 0; c < 8; ++c) red_acc[wave][h][8 * j + c] = acc[h][c];
    if (j < G) {
      red_m[wave][j] = m;
      red_l[wave][j] = l;
    }
  }
  __syncthreads();
  merge_waves<G>(red_acc, red_m, red_l, part + ((int64_t)bg * n_split + split) * G * (kD + 2));
}

// The same without grouping (G = 1), where nothing is to be shared out: the four rows that a wave instruction covers keep a state
// of their own (largest score, sum, values) until the end, so a tile needs no step across its rows.  A wave takes 16 rows at a
// time, two tiles in flight.  Every lane of a row makes its exponentials: scores are kept in units of ln 2 (the query is multiplied
// by log2(e) / sqrt(D), rounded once), so that an exponential needs no product whose rounding would have to be corrected.  In
// k_full_attn's form the few tiles of a short row waited longer for each other: 1 x 8192 rows of 8 heads in bf16 10.9 -> 9.85 us,
// in FP8 10.6 -> 9.7, 1 x 16384 in fp32 29.4 -> 28.6, 1 x 32768 in FP8 21.2 -> 19.7; 32 x 30000 in bf16 571 -> 567.
// Paged, one look-up serves both tiles: with one each, its wait came twice as often and the compiler kept fewer loads in flight (FP8
// 16 x 32768 169.2 -> 166.5 us, bf16 325.9 -> 323.2, 1 x 8192 11.7 -> 11.3).
template <typename TK, typename T, bool kPaged, bool kMayOnce>
__global__ __launch_bounds__(kAttnThreads) void k_full_attn_single(Shape s, const float* __restrict__ q,
                                                                   const TK* __restrict__ K, const T* __restrict__ V,
                                                                   int64_t stride_b, int64_t stride_h, int64_t stride_n,
                                                                   KvPage pg, const int32_t* __restrict__ seq_lens,
                                                                   float* __restrict__ part, int n_split, float) {
  constexpr double kLog2Scale = 0.08838834764831845 * 1.4426950408889634;
  constexpr float kHi = (float)kLog2Scale, kLo = (float)(kLog2Scale - (double)kHi);
  constexpr int U = 4, kRows = 4 * U;
  __shared__ float red_acc[4][1][kD];
  __shared__ float red_m[4][1], red_l[4][1];
  const int bg = blockIdx.y, b = bg / s.Hkv, g = bg % s.Hkv, split = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, rs = lane >> 4;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const int rps = rows_per_split(n, n_split);
  const int r_begin = split * rps;
  const int r_end = (r_begin + rps < n) ? r_begin + rps : n;
  if (r_begin >= n) return;
  const bool once_here = kMayOnce && outgrow_cache(s, held_rows(s, seq_lens), kD * (int)(sizeof(TK) + sizeof(T)), kKeptStreamBytes);

  float qr[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const float x = q[(int64_t)bg * kD + 8 * j + c];
    qr[c] = fmaf(x, kHi, x * kLo);
  }
  using Rows = RowMap<kPaged>;
  const TK* Kbg = K + Rows::base(b, g, stride_b, stride_h) + 8 * j;
  const T* Vbg = V + Rows::base(b, g, stride_b, stride_h) + 8 * j;

  // Rows past the end are read from the last row and weigh nothing, so no load sits behind a branch.
  struct Tile {
    Raw8<TK> k[U];                                          // my channels of row 4 u + rs
    Raw8<T> v[U];
  };
  auto clamped = [&](int r) { return r < r_end ? r : r_end - 1; };
  constexpr int kStep = 4 * kRows;                          // wave w takes tiles w, w + 4, ...
  // paged: the rows of the tiles at r0 and r0 + kStep as physical rows, in lanes 0-15 and 16-31
  auto rows_of = [&](int r0) { return kPaged ? Rows::phys(pg, b, clamped(r0 + j + (rs & 1) * kStep)) : 0; };
  auto issue = [&](auto once, Tile& t, int r0, int phys, int first_lane) {
    int64_t off[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = kPaged ? __builtin_amdgcn_ds_bpermute(4 * rs + 16 * u + 4 * first_lane, phys) : clamped(r0 + 4 * u + rs);
      off[u] = Rows::offset(pg, p, stride_b, stride_n);
    }
    load_rows<decltype(once)::value>(t.k, [&](int u) { return Kbg + off[u]; });
    load_rows<decltype(once)::value>(t.v, [&](int u) { return Vbg + off[u]; });
    __builtin_amdgcn_sched_barrier(0);                      // (moved down to their uses, the loads of one tile would wait for the other's)
  };
  float m = -INFINITY, l = 0.f, acc[8];                     // of the rows rs mod 4
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = 0.f;
  auto consume = [&](const Tile& t, int r0) {
    float sc[U], p[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float x[8];
      t.k[u].get(x);
      float a = qr[0] * x[0];
#pragma unroll
      for (int c = 1; c < 8; ++c) a = fmaf(qr[c], x[c], a);
      sc[u] = row16_butterfly_sum(a);
    }
    float mx = m;
#pragma unroll
    for (int u = 0; u < U; ++u) mx = r0 + 4 * u + rs < r_end ? fmaxf(mx, sc[u]) : mx;
    const float from = mx == -INFINITY ? 0.f : mx;          // (no row yet, or only scores of -inf: they weigh 0)
    const float alpha = __builtin_amdgcn_exp2f(m - from);   // (0 on the first tile)
    l *= alpha;
    m = mx;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float e = __builtin_amdgcn_exp2f(sc[u] - from);
      p[u] = r0 + 4 * u + rs < r_end ? e : 0.f;
      l += p[u];
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] *= alpha;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float x[8];
      t.v[u].get(x);
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[c] = fmaf(p[u], x[c], acc[c]);
    }
  };

  auto walk = [&](auto once) {
  Tile ta, tb;
  int r0 = r_begin + kRows * wave;
  int phys = rows_of(r0);
  issue(once, ta, r0, phys, 0);
  for (; r0 < r_end; r0 += 2 * kStep) {
    const int phys_next = rows_of(r0 + 2 * kStep);
    if constexpr (kPaged) __builtin_amdgcn_sched_barrier(0);      // the look-up before the rows: its wait must not include them
    issue(once, tb, r0 + kStep, phys, 16);
    consume(ta, r0);
    issue(once, ta, r0 + 2 * kStep, phys_next, 0);
    consume(tb, r0 + kStep);
    phys = phys_next;
  }
  };
  if (once_here) walk(std::true_type{});
  else walk(std::false_type{});

  // the four lane groups of the wave (one without rows: m = -inf, weight 0), then the four waves
  float mx = fmaxf(m, __shfl_xor(m, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  const float f = m == -INFINITY ? 0.f : part_weight<1>(m - mx);
  l *= f;
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    acc[c] *= f;
    acc[c] += __shfl_xor(acc[c], 16);
    acc[c] += __shfl_xor(acc[c], 32);
  }
  if (rs == 0) {
#pragma unroll
    for (int c = 0; c < 8; ++c) red_acc[wave][0][8 * j + c] = acc[c];
    if (j == 0) {
      red_m[wave][0] = mx;
      red_l[wave][0] = l;
    }
  }
  __syncthreads();
  merge_waves<1>(red_acc, red_m, red_l, part + ((int64_t)bg * n_split + split) * (kD + 2));
}

// grid B*Hq, 128 threads.  Bound by latency (1 MB of partials per 256 heads and 8 splits): the maxima and sums of all
// splits are fetched by one load each (a lane per split), the partial rows eight at a time.  Walking the splits one
// after the other took 29 us at 256 heads x 32 splits, this form 7.6 (full attention over 8 x 32K: 224 -> 207 us).
__global__ __launch_bounds__(kD) void k_full_merge(Shape s, const int32_t* __restrict__ seq_lens,
                                                   const float* __restrict__ part, int n_split,
                                                   float* __restrict__ out) {
  static_assert(kMaxSplits <= 64, "a lane per split");
  __shared__ float wgt[64], sum[64];
  const int bh = blockIdx.x, b = bh / s.Hq, h = bh % s.Hq, g = h / s.G, hg = h % s.G, c = threadIdx.x;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  if (n == 0) {
    out[(int64_t)bh * kD + c] = 0.f;
    return;
  }
  const int rps = rows_per_split(n, n_split);
  const int nv = (n + rps - 1) / rps;
  const int64_t step = (int64_t)s.G * (kD + 2);      // from one split's partials to the next one's
  const float* pb = part + ((int64_t)(b * s.Hkv + g) * n_split) * step + (int64_t)hg * (kD + 2);
  constexpr int kU = 8;
  float x[kU];
  auto fetch = [&](int sp0) {
#pragma unroll
    for (int u = 0; u < kU; ++u) x[u] = pb[(sp0 + u < nv ? sp0 + u : nv - 1) * step + c];
  };
  fetch(0);
  if (c < 64) {
    const int sp = c < nv ? c : nv - 1;
    const float m = pb[sp * step + kD];
    sum[c] = pb[sp * step + kD + 1];
    float mx = m;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) mx = fmaxf(mx, __shfl_xor(mx, d));
    wgt[c] = s.G == 1 ? part_weight<1>(m - mx) : part_weight<2>(m - mx);
  }
  __syncthreads();
  float a = 0.f, l = 0.f;
  for (int sp0 = 0;;) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      if (sp0 + u < nv) {
        a = fmaf(x[u], wgt[sp0 + u], a);
        l = fmaf(sum[sp0 + u], wgt[sp0 + u], l);
      }
    }
    sp0 += kU;
    if (sp0 >= nv) break;
    fetch(sp0);
  }
  out[(int64_t)bh * kD + c] = a / l;
}

template <typename TK, typename T>
static hipError_t launch_full_t(const Shape& s, const float* q, const KvView& kv, float* part, int n_split,
                                hipStream_t st) {
  const dim3 grid(n_split, s.B * s.Hkv), block(kAttnThreads);
  const float scale = 0.08838834764831845f;
  // (the kernels ask how many rows are held; fp32 rows: a lane's eight channels are two loads, which would fetch the line twice)
  const bool once = sizeof(TK) < 4 && (int64_t)s.B * s.Hkv * s.Lcap * kD * (int64_t)(sizeof(TK) + sizeof(T)) > kKeptStreamBytes;
#define LFPS_LAUNCH_FULL_P(KERNEL, PAGED, ONCE, ...)                                                                    \
  hipLaunchKernelGGL((KERNEL<TK, T, ##__VA_ARGS__, PAGED, ONCE>), grid, block, 0, st, s, q, (const TK*)kv.k,             \
                     (const T*)kv.v, kv.stride_b, kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, part, n_split, scale)
#define LFPS_LAUNCH_FULL(KERNEL, ...)                                                   \
  if (kv.page.table) {                                                                  \
    if (once) LFPS_LAUNCH_FULL_P(KERNEL, true, sizeof(TK) < 4, ##__VA_ARGS__);          \
    else LFPS_LAUNCH_FULL_P(KERNEL, true, false, ##__VA_ARGS__);                        \
  } else {                                                                              \
    if (once) LFPS_LAUNCH_FULL_P(KERNEL, false, sizeof(TK) < 4, ##__VA_ARGS__);         \
    else LFPS_LAUNCH_FULL_P(KERNEL, false, false, ##__VA_ARGS__);                       \
  }
  switch (s.G) {
    case 1: LFPS_LAUNCH_FULL(k_full_attn_single); break;
    case 2: LFPS_LAUNCH_FULL(k_full_attn, 2); break;
    case 4: LFPS_LAUNCH_FULL(k_full_attn, 4); break;
    default: return hipErrorInvalidValue;
  }
#undef LFPS_LAUNCH_FULL
#undef LFPS_LAUNCH_FULL_P
  return hipGetLastError();
}

hipError_t launch_full_attn(const Shape& s, int dtype, const float* q, const KvView& kv, float* part, int n_split,
                            hipStream_t st) {
  if (dtype == LFPS_BF16 && kv.k_fp8 && kv.v_fp8) return launch_full_t<uint8_t, uint8_t>(s, q, kv, part, n_split, st);
  if (dtype == LFPS_BF16 && kv.k_fp8) return launch_full_t<uint8_t, uint16_t>(s, q, kv, part, n_split, st);
  if (dtype == LFPS_BF16 && kv.v_fp8) return launch_full_t<uint16_t, uint8_t>(s, q, kv, part, n_split, st);
  if (dtype == LFPS_F16) return launch_full_t<_Float16, _Float16>(s, q, kv, part, n_split, st);
  return dtype == LFPS_BF16 ? launch_full_t<uint16_t, uint16_t>(s, q, kv, part, n_split, st)
                            : launch_full_t<float, float>(s, q, kv, part, n_split, st);
}

hipError_t launch_full_merge(const Shape& s, const int32_t* seq_lens, const float* part, int n_split, float* out,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_full_merge, dim3(s.B * s.Hq), dim3(kD), 0, st, s, seq_lens, part, n_split, out);
  return hipGetLastError();
}

}  // namespace lfps
