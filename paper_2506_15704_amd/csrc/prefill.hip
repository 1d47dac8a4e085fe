// What prefill hands to decode: the score tables from the last s prefill queries (Eq. 4), their statistics, and the
// priors of the head-sparsity test (Sec. 4.2 "Prefilling", last paragraph).
//
// Eq. 4 needs, for every one of s queries and every head, the softmax of its scores over all rows it sees.  One query
// at a time that is s passes over K (16-bit keys at 8 groups x 32K rows: 14 us of scoring that writes every score, and
// 30 us of softmax and accumulation that reads and writes scores and tables, per query: 1.4 ms for s = 32).  K is the
// same for all of them, so here a wave keeps 128 rows of K in registers as MFMA operands and walks the queries:
//   k_hist_stats   per (query, head) the largest score and the sum of exponentials, in one pass over K;
//   k_hist_apply   the scores once more (the same bits), the weights, and the sums over the queries, which never leave
//                  registers: every table entry is written once.
// Two passes over K are needed because a weight needs the sum over all rows; storing the scores between them would
// cost 4 bytes per row, query and head (8.6 times the bytes of a second pass over bf16 keys at s = 32, G = 4).
// The kernels are bound by the matrix and vector units (per 64 rows and query 16 MFMAs of 16 cycles, and about as much
// time again in vector instructions, most of them the exponentials and the fp64 sums): 32 queries of 8 groups x 32K rows
// take 48 + 59 us, beside 1.42 ms one query at a time.
#include "lfps_internal.h"
#include "score_mfma.h"

#include <float.h>

#include <type_traits>

namespace lfps {

constexpr int kHistWaves = 8;          // one workgroup per CU: the query operands fill its LDS, the rows its registers
constexpr int kHistSub = 8;            // 16-row sub-tiles a wave holds: 128 rows
constexpr int kHistRows = 16 * kHistSub;
constexpr float kNoScore = -FLT_MAX;   // stands for "row not seen"
constexpr float kLeastMax = -1.7e38f;  // the largest score is taken as at least this: a row not seen weighs 0 beside any

__host__ __device__ constexpr int hist_lds(int nq) { return nq * 4 * 64 * 16; }   // bytes of the operands of nq queries

// MFMA A operands (layout of load_query_operand) of nq queries for the heads of group (b, g), to LDS:
// entry (jq * 4 + kk) * 64 + lane.  A thread makes the three terms (and the zero row) of 8 channels of one head.
// Returns true if it met an element beyond the fp16 range.
template <int G, typename Op>
__device__ __forceinline__ bool stage_hist_operands(Op* lds, const float* __restrict__ q0, int64_t q_stride,
                                                    int64_t head0, int nq) {
  bool clipped = false;
  for (int u = threadIdx.x; u < nq * 64; u += kHistWaves * 64) {
    const int jq = u >> 6, h = (u >> 4) & 3, kk = (u >> 2) & 3, kb = u & 3;
    Op* e = lds + (jq * 4 + kk) * 64 + kb * 16 + 4 * h;
    const float4* p = reinterpret_cast<const float4*>(q0 + jq * q_stride + (head0 + (h < G ? h : 0)) * kD) + 2 * (kk + 4 * kb);
    const float4 lo = p[0], hi = p[1];
    float f[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    if constexpr (Split3<Op>::kHalf) {
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        if (fabsf(f[c]) > 65504.0f) {
          clipped |= h < G;
          f[c] = copysignf(65504.0f, f[c]);
        }
      }
    }
    Op term[3];
    Split3<Op>::all(f, term);
    const uint32_t live = h < G ? ~0u : 0u;                // (by bits: from a choice the compiler makes two branches)
#pragma unroll
    for (int t = 0; t < 3; ++t) e[t] = __builtin_bit_cast(Op, __builtin_bit_cast(u32x4, term[t]) & live);
    e[3] = Op{};
  }
  return clipped;
}

// NT sub-tiles of K rows as MFMA operands: lane (j, kb) holds its channels of the rows base + 16 t + j.  Rows past the
// sequence read its last row.
template <bool kPaged, int kKind, int NT>
struct HistTile {
  using Op = typename KSub<kKind>::Operand;
  Op x[NT][4];
  __device__ __forceinline__ void load(const char* Kbg, const KvPage& pg, int b, int64_t stride_b, int64_t stride_n,
                                       int base, int n, int j, int kb) {
    using Rows = RowMap<kPaged>;
    KSub<kKind> raw[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int row = base + 16 * t + j;
      const int p = Rows::phys(pg, b, row < n ? row : n - 1);
      raw[t].load_row(Kbg + Rows::offset(pg, p, stride_b, stride_n) * KSub<kKind>::kElemBytes, kb);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) x[t][kk] = raw[t].operand(kk);
  }
  // the same past the caches; turn: StreamTile's piece of LDS of this wave
  __device__ __forceinline__ void load_once(const char* Kbg, const KvPage& pg, int b, int64_t stride_b, int64_t stride_n,
                                            int base, int n, int lane, u32x4* turn) {
    using Rows = RowMap<kPaged>;
    static_assert(NT % 4 == 0, "whole stream tiles");
    StreamTile<kKind> raw[NT / 4];
#pragma unroll
    for (int u = 0; u < NT / 4; ++u) {
      const int row = base + kRowsPerWaveIter * u + lane;
      raw[u].fetch(Kbg, Rows::phys(pg, b, row < n ? row : n - 1), lane,
                   [&](int p) { return Rows::offset(pg, p, stride_b, stride_n) * KSub<kKind>::kElemBytes; });
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const KSub<kKind> sub = raw[t / 4].sub(t % 4, turn, lane);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) x[t][kk] = sub.operand(kk);
    }
  }
  // v[t] = q . K (not yet divided by sqrt(D)) of my row of sub-tile t for head kb and the query whose operands start at a
  __device__ __forceinline__ void dots(const Op* a, int lane, float (&v)[NT]) const {
    Op A[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) A[kk] = a[kk * 64 + lane];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) acc = mfma16(A[kk], x[t][kk], acc);
      v[t] = Split3<Op>::sum(acc);
    }
  }
};

// Tiles [lo, hi) of `tiles` that fall to wave w of `waves`: contiguous runs.
__device__ __forceinline__ void wave_run(int tiles, int w, int waves, int& lo, int& hi) {
  const int per = (tiles + waves - 1) / waves;
  lo = w * per < tiles ? w * per : tiles;
  hi = lo + per < tiles ? lo + per : tiles;
}

// grid (blocks per group, B*Hkv).  Queries j0 .. j0 + nq - 1 (j = 1: the most recent); query j sees the offloaded rows
// [n_sink, n - j + 1).  part_m / part_l [bg, block, jq, h]: the largest q . K and the sum of the exponentials relative
// to it over the rows of the block (kLeastMax and 0 when it has none).  dots (or NULL; one query only): every q . K,
// [B, Hq, stride].
// kMayOnce: rows past the caches (StreamTile; its LDS lies behind the operands) where the requests hold more than kept_bytes of
// them, see stats_kept_bytes.
template <int G, bool kPaged, int kKind, bool kMayOnce>
__global__ __launch_bounds__(kHistWaves * 64) void k_hist_stats(
    Shape s, const float* __restrict__ q0, int64_t q_stride, int j0, int nq, const void* __restrict__ K,
    int64_t stride_b, int64_t stride_h, int64_t stride_n, KvPage pg, const int32_t* __restrict__ seq_lens,
    float* __restrict__ part_m, double* __restrict__ part_l, float* __restrict__ dots, int64_t dots_stride,
    int32_t* __restrict__ flags, float kept_bytes) {
  using Tile = HistTile<kPaged, kKind, kHistSub>;
  using Op = typename Tile::Op;
  extern __shared__ char lds_raw[];
  Op* ops = reinterpret_cast<Op*>(lds_raw);
  __shared__ float wm[kHistWaves][kHistBatch][4];
  __shared__ double wl[kHistWaves][kHistBatch][4];
  const int bg = blockIdx.y, b = bg / s.Hkv, g = bg % s.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, kb = lane >> 4;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const float held = kMayOnce ? held_rows(s, seq_lens) : 0.f;
  report_q_range(stage_hist_operands<G>(ops, q0, q_stride, (int64_t)b * s.Hq + (int64_t)g * G, nq), flags);
  for (int e = tid; e < kHistWaves * kHistBatch * 4; e += kHistWaves * 64) {
    (&wm[0][0][0])[e] = kLeastMax;
    (&wl[0][0][0])[e] = 0.0;
  }
  const bool once = kMayOnce && outgrow_cache(s, held, kD * KSub<kKind>::kElemBytes, kept_bytes);
  __syncthreads();
  const char* Kbg = static_cast<const char*>(K) + RowMap<kPaged>::base(b, g, stride_b, stride_h) * KSub<kKind>::kElemBytes;
  float* my_dots = dots && kb < G ? dots + ((int64_t)b * s.Hq + (int64_t)g * G + kb) * dots_stride : nullptr;
  int lo, hi;
  wave_run((n + kHistRows - 1) / kHistRows, blockIdx.x * kHistWaves + wave, gridDim.x * kHistWaves, lo, hi);
  for (int tile = lo; tile < hi; ++tile) {
    const int base = tile * kHistRows;
    Tile T;
    if (kMayOnce && once)                                  // (a copy of the loop each: 1.5 us slower at 64 groups x 17K rows)
      T.load_once(Kbg, pg, b, stride_b, stride_n, base, n, lane,
                  reinterpret_cast<u32x4*>(lds_raw + hist_lds(nq)) + wave * StreamTile<kKind>::kLdsChunks);
    else
      T.load(Kbg, pg, b, stride_b, stride_n, base, n, j, kb);
    // a tile of which every query sees every row needs no masks (wave-uniform)
    const bool whole = base >= s.n_sink && base + kHistRows <= n - (j0 + nq - 1) + 1;
    auto walk = [&](auto masked) {
      for (int jq = 0; jq < nq; ++jq) {
        float v[kHistSub];
        T.dots(ops + jq * 256, lane, v);
        if constexpr (decltype(masked)::value) {
          const int seen = n - (j0 + jq) + 1;
#pragma unroll
          for (int t = 0; t < kHistSub; ++t) {
            const int row = base + 16 * t + j;
            v[t] = row >= s.n_sink && row < seen ? v[t] : kNoScore;
          }
        }
        float mx = v[0];
#pragma unroll
        for (int t = 1; t < kHistSub; ++t) mx = fmaxf(mx, v[t]);
        mx = row16_max(mx);
        const float m_old = wm[wave][jq][kb];
        const float m = fmaxf(m_old, mx);
        double l = 0.0;
#pragma unroll
        for (int t = 0; t < kHistSub; ++t) l += (double)exp_below<true>(v[t] - m);
        l = row16_sum(l);
        if (j == 0) {
          wl[wave][jq][kb] = wl[wave][jq][kb] * (double)exp_below<true>(m_old - m) + l;
          wm[wave][jq][kb] = m;
        }
        if (my_dots) {
#pragma unroll
          for (int t = 0; t < kHistSub; ++t) {
            const int row = base + 16 * t + j;
            if (row < n) my_dots[row] = v[t];
          }
        }
      }
    };
    if (whole) walk(std::false_type{});
    else walk(std::true_type{});
    wave_lds_order();                                      // wm of this tile before the other lanes read it in the next
  }
  __syncthreads();
  for (int e = tid; e < nq * G; e += kHistWaves * 64) {
    const int jq = e / G, h = e % G;
    float m = kLeastMax;
#pragma unroll
    for (int w = 0; w < kHistWaves; ++w) m = fmaxf(m, wm[w][jq][h]);
    double l = 0.0;
#pragma unroll
    for (int w = 0; w < kHistWaves; ++w) l += wl[w][jq][h] * (double)exp_below<true>(wm[w][jq][h] - m);
    const int64_t o = ((int64_t)bg * gridDim.x + blockIdx.x) * (kHistBatch * G) + e;
    part_m[o] = m;
    part_l[o] = l;
  }
}

// The partials of one (query, head), merged by kPer neighbouring lanes (sub = 0 .. kPer - 1): the largest dot
// product, and the factor 1 / (2 s (1 - gamma) sum) that turns an exponential into a table contribution.
template <int kPer>
__device__ __forceinline__ void merge_hist(const float* part_m, const double* part_l, int64_t o, int64_t step, int blocks,
                                           int sub, double gamma, int n_queries, float& m, double& norm) {
  m = kLeastMax;
#pragma unroll 8
  for (int k = sub; k < blocks; k += kPer) m = fmaxf(m, part_m[o + k * step]);
#pragma unroll
  for (int d = 1; d < kPer; d <<= 1) m = fmaxf(m, __shfl_xor(m, d));
  double l = 0.0;
#pragma unroll 8
  for (int k = sub; k < blocks; k += kPer) l += part_l[o + k * step] * (double)exp_below<true>(part_m[o + k * step] - m);
#pragma unroll
  for (int d = 1; d < kPer; d <<= 1) l += __shfl_xor(l, d);
  norm = l > 0.0 ? 1.0 / (2.0 * (double)n_queries * (1.0 - gamma) * l) : 0.0;
}

// e * norm rounded once to fp32 (norm = hi + lo).
__device__ __forceinline__ float weigh(float e, float hi, float lo) { return fmaf(e, hi, e * lo); }

// The same grid and queries.  Adds  w_j(i) / (2 s (1 - gamma))  to the vertical table at i and to the slash table at
// i + j - 1, for all nq queries at once; the first batch (j0 = 1) writes the tables whole (zeros past the sequence and
// in the lower half of the slash frame), later batches add to them.
// The slash sums need no scatter: walked from the oldest query of the batch to the newest, with the running sums moved
// one row up before each query's weights are added, row p ends with sum_i w_{j0 + i}(p - i), which belongs at slash
// position p + j0 - 1.  Lanes are consecutive rows, so the move is a rotation inside 16 lanes; the value that enters a
// tile at its first row was left per query by the tile before (carry).  A wave starts its run of tiles with the 32
// rows before it, for their carries alone (a batch reaches back at most 31 rows).
template <int G, bool kPaged, int kKind>
__global__ __launch_bounds__(kHistWaves * 64) void k_hist_apply(
    Shape s, float* __restrict__ tab_ver, float* __restrict__ tab_sla, const float* __restrict__ q0, int64_t q_stride,
    int j0, int nq, const void* __restrict__ K, int64_t stride_b, int64_t stride_h, int64_t stride_n, KvPage pg,
    const int32_t* __restrict__ seq_lens, const float* __restrict__ part_m, const double* __restrict__ part_l,
    double gamma, int n_queries) {
  using Op = typename KSub<kKind>::Operand;
  extern __shared__ char lds_raw[];
  Op* ops = reinterpret_cast<Op*>(lds_raw);
  __shared__ float ref[kHistBatch][4][3];                  // largest dot product, factor as a pair of floats
  __shared__ float carry[kHistWaves][kHistBatch][4];
  const int bg = blockIdx.y, b = bg / s.Hkv, g = bg % s.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, kb = lane >> 4;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  (void)stage_hist_operands<G>(ops, q0, q_stride, (int64_t)b * s.Hq + (int64_t)g * G, nq);   // (k_hist_stats reported the range)
  {
    static_assert(kHistWaves * 64 == kHistBatch * 4 * 4, "four lanes per query and head");
    const int jq = tid >> 4, h = (tid >> 2) & 3, sub = tid & 3;
    if (jq < nq && h < G) {                                // uniform over the four lanes
      float m;
      double norm;
      merge_hist<4>(part_m, part_l, (int64_t)bg * gridDim.x * (kHistBatch * G) + jq * G + h, kHistBatch * G, gridDim.x,
                    sub, gamma, n_queries, m, norm);
      const float hi = (float)norm;
      ref[jq][h][0] = m;
      ref[jq][h][1] = hi;
      ref[jq][h][2] = (float)(norm - (double)hi);
    }
  }
  for (int e = tid; e < kHistWaves * kHistBatch * 4; e += kHistWaves * 64) (&carry[0][0][0])[e] = 0.f;
  __syncthreads();

  const char* Kbg = static_cast<const char*>(K) + RowMap<kPaged>::base(b, g, stride_b, stride_h) * KSub<kKind>::kElemBytes;
  const int64_t bh = (int64_t)b * s.Hq + (int64_t)g * G + (kb < G ? kb : 0);
  float* ver = tab_ver + bh * s.Lcap;
  float* sla = tab_sla + bh * 2 * s.Lcap;                  // position p of an untouched table is slot Lcap + p
  float(*my_carry)[4] = carry[wave];
  const int kh = kb < G ? kb : 0;
  auto walk = [&](auto& T, int base, auto& av, auto& as, auto masked) {
    constexpr int NT = sizeof(av) / sizeof(float);
    float cin = 0.f;                                       // what enters at row `base` from the row before
    for (int jq = nq - 1; jq >= 0; --jq) {
      float v[NT];
      T.dots(ops + jq * 256, lane, v);
      const float m = ref[jq][kh][0], hi = ref[jq][kh][1], lo = ref[jq][kh][2];
      const float next_cin = my_carry[jq][kb];
      float up[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) up[t] = row16_rotate<1>(as[t]);
#pragma unroll
      for (int t = NT - 1; t >= 0; --t) {
        if constexpr (decltype(masked)::value) {
          const int row = base + 16 * t + j;
          v[t] = row >= s.n_sink && row < n - (j0 + jq) + 1 ? v[t] : kNoScore;
        }
        const float w = weigh(exp_below<true>(v[t] - m), hi, lo);
        av[t] += w;
        const float moved = j != 0 ? up[t] : (t == 0 ? cin : up[t > 0 ? t - 1 : 0]);
        as[t] = moved + w;
      }
      if (j == 15) my_carry[jq][kb] = as[NT - 1];
      cin = next_cin;
    }
    wave_lds_order();                                      // the carries before the other lanes read them for the next rows
  };
  auto walk_rows = [&](auto& T, int base, auto& av, auto& as) {
    constexpr int NT = sizeof(av) / sizeof(float);
    if (base >= s.n_sink && base + 16 * NT <= n - (j0 + nq - 1) + 1) walk(T, base, av, as, std::false_type{});
    else walk(T, base, av, as, std::true_type{});
  };
  const int tiles = (n + kHistRows - 1) / kHistRows;
  int lo, hi;
  wave_run(tiles, blockIdx.x * kHistWaves + wave, gridDim.x * kHistWaves, lo, hi);
  if (lo < hi && lo > 0 && nq > 1) {
    HistTile<kPaged, kKind, 2> T;
    const int base = lo * kHistRows - 32;
    T.load(Kbg, pg, b, stride_b, stride_n, base, n, j, kb);
    float av[2] = {0.f, 0.f}, as[2] = {0.f, 0.f};
    walk_rows(T, base, av, as);
  }
  const bool first = j0 == 1;
  for (int tile = lo; tile < hi; ++tile) {
    const int base = tile * kHistRows;
    HistTile<kPaged, kKind, kHistSub> T;
    T.load(Kbg, pg, b, stride_b, stride_n, base, n, j, kb);
    float av[kHistSub], as[kHistSub];
#pragma unroll
    for (int t = 0; t < kHistSub; ++t) av[t] = as[t] = 0.f;
    walk_rows(T, base, av, as);
    if (kb < G) {
#pragma unroll
      for (int t = 0; t < kHistSub; ++t) {
        const int row = base + 16 * t + j;
        const int pos = row + j0 - 1;
        if (first) {
          if (row < s.Lcap) {                              // past the sequence the sums are zero
            ver[row] = av[t];
            sla[s.Lcap + row] = as[t];
            sla[row] = 0.f;
          }
        } else {
          if (row < n) ver[row] += av[t];
          if (pos < n) sla[s.Lcap + pos] += as[t];
        }
      }
    }
  }
  if (first) {
    for (int h = 0; h < G; ++h) {
      float* vh = tab_ver + ((int64_t)b * s.Hq + (int64_t)g * G + h) * s.Lcap;
      float* sh = tab_sla + ((int64_t)b * s.Hq + (int64_t)g * G + h) * 2 * s.Lcap;
      for (int i = tiles * kHistRows + blockIdx.x * kHistWaves * 64 + tid; i < s.Lcap; i += gridDim.x * kHistWaves * 64) {
        vh[i] = 0.f;
        sh[s.Lcap + i] = 0.f;
        sh[i] = 0.f;
      }
    }
  }
}

// M1..M4 of the vertical and of the slash entries of a workgroup (256 threads, U positions each, those with in[u]), then
// the smallest and the negated largest of both, to out[0:12].
template <int U>
__device__ __forceinline__ void moments_of_chunk(const float (&xv)[U], const float (&xs)[U], const bool (&in)[U],
                                                 double* __restrict__ out) {
  __shared__ double red[4][12];
  const int tid = threadIdx.x;
  double m[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  float e[4] = {INFINITY, INFINITY, INFINITY, INFINITY};
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (!in[u]) continue;
    const double a = xv[u], c = xs[u];
    m[0] += a; m[1] += a * a; m[2] += a * a * a; m[3] += a * a * a * a;
    m[4] += c; m[5] += c * c; m[6] += c * c * c; m[7] += c * c * c * c;
    e[0] = fminf(e[0], xv[u]); e[1] = fminf(e[1], -xv[u]);
    e[2] = fminf(e[2], xs[u]); e[3] = fminf(e[3], -xs[u]);
  }
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    m[p] = row16_sum(m[p]);
    m[p] += __shfl_xor(m[p], 16);
    m[p] += __shfl_xor(m[p], 32);
  }
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    e[p] = -row16_max(-e[p]);
    e[p] = fminf(e[p], __shfl_xor(e[p], 16));
    e[p] = fminf(e[p], __shfl_xor(e[p], 32));
  }
  if ((tid & 63) == 0) {
#pragma unroll
    for (int p = 0; p < 8; ++p) red[tid >> 6][p] = m[p];
#pragma unroll
    for (int p = 0; p < 4; ++p) red[tid >> 6][8 + p] = (double)e[p];
  }
  __syncthreads();
  if (tid < 12) {
    double t = red[0][tid];
    for (int w = 1; w < 4; ++w) t = tid < 8 ? t + red[w][tid] : fmin(t, red[w][tid]);
    out[tid] = t;
  }
}

// One query (s = 1): its dot products are few enough to store (4 bytes per row and head beside 2 D / G of K), so the
// second pass over K is replaced by this one over them.  Vertical and slash table are equal then.  Writes the tables
// whole, and the moments of its rows as k_table_moments does.  grid (chunks, B*Hq), 256 threads.
constexpr int kMomentRows = 2048;
__global__ __launch_bounds__(256) void k_hist_apply_one(Shape s, float* __restrict__ tab_ver, float* __restrict__ tab_sla,
                                                        const float* __restrict__ dots, int64_t dots_stride,
                                                        const int32_t* __restrict__ seq_lens,
                                                        const float* __restrict__ part_m,
                                                        const double* __restrict__ part_l, int blocks, double gamma,
                                                        double* __restrict__ part) {
  const int bh = blockIdx.y, b = bh / s.Hq, h = bh % s.Hq, g = h / s.G, tid = threadIdx.x;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  constexpr int U = kMomentRows / 256;
  float x[U];
  bool in[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = blockIdx.x * kMomentRows + u * 256 + tid;
    in[u] = i >= s.n_sink && i < n;
    x[u] = in[u] ? dots[(int64_t)bh * dots_stride + i] : kNoScore;
  }
  float m;
  double norm;
  merge_hist<64>(part_m, part_l, ((int64_t)b * s.Hkv + g) * blocks * (kHistBatch * s.G) + h % s.G, kHistBatch * s.G,
                 blocks, tid & 63, gamma, 1, m, norm);
  const float hi = (float)norm, lo = (float)(norm - (double)hi);
  float* ver = tab_ver + (int64_t)bh * s.Lcap;
  float* sla = tab_sla + (int64_t)bh * 2 * s.Lcap;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = blockIdx.x * kMomentRows + u * 256 + tid;
    x[u] = in[u] ? weigh(exp_below<true>(x[u] - m), hi, lo) : 0.f;
    if (i < s.Lcap) {
      ver[i] = x[u];
      sla[s.Lcap + i] = x[u];
      sla[i] = 0.f;
    }
  }
  moments_of_chunk<U>(x, x, in, part + ((int64_t)bh * gridDim.x + blockIdx.x) * 12);
}

// ----------------------------------------------------------------------------- statistics of a fresh table
// Raw moments and extremes of both tables over the offloaded positions, one partial per chunk of kMomentRows rows
// (one workgroup per head took 28 us at 32 heads x 32K entries: 32 of 256 CUs busy).  grid (chunks, B*Hq).
__global__ __launch_bounds__(256) void k_table_moments(Shape s, const float* __restrict__ tab_ver,
                                                       const float* __restrict__ tab_sla,
                                                       const int32_t* __restrict__ seq_lens, double* __restrict__ part) {
  const int bh = blockIdx.y, b = bh / s.Hq, tid = threadIdx.x;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const float* ver = tab_ver + (int64_t)bh * s.Lcap;
  const float* sla = tab_sla + (int64_t)bh * 2 * s.Lcap + s.Lcap;
  constexpr int U = kMomentRows / 256;
  float xv[U], xs[U];
  bool in[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = blockIdx.x * kMomentRows + u * 256 + tid;
    in[u] = i >= s.n_sink && i < n;
    xv[u] = in[u] ? ver[i] : 0.f;
    xs[u] = in[u] ? sla[i] : 0.f;
  }
  moments_of_chunk<U>(xv, xs, in, part + ((int64_t)bh * gridDim.x + blockIdx.x) * 12);
}

// Scale 1, update count 0, raw moments and flat marks from the partials.  grid B*Hq, 192 threads: sixteen per value.
__global__ __launch_bounds__(192) void k_table_state(Shape s, const double* __restrict__ part, int chunks,
                                                     double* __restrict__ state, const int32_t* __restrict__ seq_lens) {
  __shared__ double tot[12];
  const int bh = blockIdx.x, b = bh / s.Hq, v = threadIdx.x >> 4, sub = threadIdx.x & 15;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const double* p = part + (int64_t)bh * chunks * 12 + v;
  double t = v < 8 ? 0.0 : INFINITY;
#pragma unroll 4
  for (int c = sub; c < chunks; c += 16) t = v < 8 ? t + p[c * 12] : fmin(t, p[c * 12]);
#pragma unroll
  for (int d = 1; d < 16; d <<= 1) {
    const double o = __shfl_xor(t, d);
    t = v < 8 ? t + o : fmin(t, o);
  }
  if (sub == 0) tot[v] = t;
  __syncthreads();
  double* st = state + (int64_t)bh * kTableStateDoubles;
  if (threadIdx.x < 8) st[TS_MV + threadIdx.x] = tot[threadIdx.x];   // both tables' moments lie side by side
  if (threadIdx.x == 0) {
    st[TS_G] = 1.0;
    st[TS_CNT] = 0.0;
    st[TS_FLAT_V] = -tot[9] > tot[8] ? 0.0 : 1.0;                    // every entry equal: no pattern
    st[TS_FLAT_S] = -tot[11] > tot[10] ? 0.0 : 1.0;
    st[TS_FLAT_N] = (double)(n - s.n_sink > 0 ? n - s.n_sink : 0);
  }
}
static_assert(TS_MS == TS_MV + 4, "k_table_state writes both sets of moments in a row");

// ----------------------------------------------------------------------------- prefill priors
// K mean, V mean and the variance of the scaled scores of the given query over the offloaded rows, from one pass over
// K and V (three passes before, the means by one workgroup per KV group: 8 of 256 CUs at B = 1).  Bound by the bytes of
// K and V: 34 + 8 us at 8 groups x 32K bf16 rows (134 MB), 600 us before.  grid (splits, B*Hkv), 256 threads; 16 lanes per row, 8 channels each, two 16-row tiles per wave in flight.
// Per (bg, split) a partial: 128 sums of K, 128 of V, then (rows, mean, sum of squared deviations) of every head's
// scores; the means and deviations of parts are merged exactly (no difference of large sums).
constexpr int kPriorThreads = 256;
__host__ __device__ constexpr int prior_partial(int G) { return 2 * kD + 3 * G; }   // doubles

__device__ __forceinline__ void merge_moments(double& n, double& mean, double& m2, double n2, double mean2, double m22) {
  if (n2 <= 0.0) return;
  const double t = n + n2, d = mean2 - mean;
  mean += d * (n2 / t);
  m2 += m22 + d * d * (n * n2 / t);
  n = t;
}

template <typename TK, typename T, int G, bool kPaged>
__global__ __launch_bounds__(kPriorThreads) void k_prior_partials(Shape s, const float* __restrict__ q,
                                                                  const TK* __restrict__ K, const T* __restrict__ V,
                                                                  int64_t stride_b, int64_t stride_h, int64_t stride_n,
                                                                  KvPage pg, const int32_t* __restrict__ seq_lens,
                                                                  double* __restrict__ part, float scale,
                                                                  int32_t* __restrict__ flags) {
  __shared__ double red[4][2 * kD];
  __shared__ double hist[4][4][G][3];
  const int bg = blockIdx.y, b = bg / s.Hkv, g = bg % s.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = lane & 15, rs = lane >> 4;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const int rows = n - s.n_sink > 0 ? n - s.n_sink : 0;
  const int per = (((rows + (int)gridDim.x - 1) / (int)gridDim.x) + 15) & ~15;
  const int r_begin = s.n_sink + blockIdx.x * per;
  const int r_end = r_begin + per < n ? r_begin + per : n;

  float qr[G][8];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float* qh = q + ((int64_t)b * s.Hq + (int64_t)g * G + h) * kD + 8 * j;
#pragma unroll
    for (int c = 0; c < 8; ++c) qr[h][c] = qh[c];
  }
  if constexpr (std::is_same<TK, _Float16>::value) {       // as in the scoring kernels: beyond the fp16 range, clamped
    bool clipped = false;
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        if (fabsf(qr[h][c]) > 65504.0f) {
          clipped = true;
          qr[h][c] = copysignf(65504.0f, qr[h][c]);
        }
      }
    report_q_range(clipped, flags);
  }
  using Rows = RowMap<kPaged>;
  const TK* Kbg = K + Rows::base(b, g, stride_b, stride_h) + 8 * j;
  const T* Vbg = V + Rows::base(b, g, stride_b, stride_h) + 8 * j;
  constexpr int U = 4;
  struct Tile {
    Raw8<TK> k[U];
    Raw8<T> v[U];
  };
  auto issue = [&](Tile& t, int r0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int r = r0 + 4 * u + rs;
      r = r < r_end ? r : r_end - 1;
      const int64_t off = Rows::offset(pg, Rows::phys(pg, b, r), stride_b, stride_n);
      t.k[u].load(Kbg + off);
      t.v[u].load(Vbg + off);
    }
  };
  float ks[8], vs[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) ks[c] = vs[c] = 0.f;
  double shift = 0.0, d1 = 0.0, d2 = 0.0, cnt = 0.0;      // of head j (lanes j < G), around the first score seen
  auto consume = [&](const Tile& t, int r0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool ok = r0 + 4 * u + rs < r_end;
      float kx[8], vx[8];
      t.k[u].get(kx);
      t.v[u].get(vx);
      float x = 0.f;
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float a = qr[h][0] * kx[0];
#pragma unroll
        for (int c = 1; c < 8; ++c) a = fmaf(qr[h][c], kx[c], a);
        a = row16_sum(a);
        x = j == h ? a : x;
      }
      if (ok) {
        const double sc = (double)(x * scale);
        if (cnt == 0.0) shift = sc;
        const double d = sc - shift;
        d1 += d;
        d2 += d * d;
        cnt += 1.0;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          ks[c] += kx[c];
          vs[c] += vx[c];
        }
      }
    }
  };
  if (r_begin < r_end) {
    Tile ta, tb;
    int r0 = r_begin + 16 * wave;
    issue(ta, r0);
    for (; r0 < r_end; r0 += 128) {
      issue(tb, r0 + 64);
      consume(ta, r0);
      issue(ta, r0 + 128);
      consume(tb, r0 + 64);
    }
  }
  // the four row slots of a wave, then the four waves
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    double a = ks[c], v = vs[c];
    a += __shfl_xor(a, 16);
    v += __shfl_xor(v, 16);
    a += __shfl_xor(a, 32);
    v += __shfl_xor(v, 32);
    if (rs == 0) {
      red[wave][8 * j + c] = a;
      red[wave][kD + 8 * j + c] = v;
    }
  }
  if (j < G) {
    hist[wave][rs][j][0] = cnt;
    hist[wave][rs][j][1] = cnt > 0.0 ? shift + d1 / cnt : 0.0;
    hist[wave][rs][j][2] = cnt > 0.0 ? d2 - d1 * d1 / cnt : 0.0;
  }
  __syncthreads();
  double* po = part + ((int64_t)bg * gridDim.x + blockIdx.x) * prior_partial(G);
  po[tid] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);      // kPriorThreads == 2 kD
  if (tid < G) {
    double c = 0.0, mean = 0.0, m2 = 0.0;
    for (int w = 0; w < 4; ++w)
      for (int r = 0; r < 4; ++r) merge_moments(c, mean, m2, hist[w][r][tid][0], hist[w][r][tid][1], hist[w][r][tid][2]);
    po[2 * kD + 3 * tid] = c;
    po[2 * kD + 3 * tid + 1] = mean;
    po[2 * kD + 3 * tid + 2] = m2;
  }
}

// grid B*Hkv, 1024 threads: the partials of a group.  Four threads per channel take every fourth split; wave h merges
// the scores of head h.
__global__ __launch_bounds__(1024) void k_prior_final(Shape s, const float* __restrict__ q,
                                                      const int32_t* __restrict__ seq_lens,
                                                      const double* __restrict__ part, int splits,
                                                      float* __restrict__ kbar, float* __restrict__ vbar,
                                                      float* __restrict__ sigma2_hat) {
  __shared__ double red[4][2 * kD];
  const int bg = blockIdx.x, b = bg / s.Hkv, g = bg % s.Hkv, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const int cnt = n - s.n_sink;
  const int stride = prior_partial(s.G);
  const double* p = part + (int64_t)bg * splits * stride;
  const int c = tid & (2 * kD - 1);
  double t = 0.0;
#pragma unroll 8
  for (int k = tid / (2 * kD); k < splits; k += 4) t += p[(int64_t)k * stride + c];
  red[tid / (2 * kD)][c] = t;
  __syncthreads();
  if (tid < 2 * kD) {
    t = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
    (c < kD ? kbar : vbar)[(int64_t)bg * kD + (c & (kD - 1))] = cnt > 0 ? (float)(t / (double)cnt) : 0.f;
  }
  if (wave < s.G) {
    const int64_t bh = (int64_t)b * s.Hq + (int64_t)g * s.G + wave;
    double rows = 0.0, mean = 0.0, m2 = 0.0;
    for (int k = lane; k < splits; k += 64) {
      const double* h = p + (int64_t)k * stride + 2 * kD + 3 * wave;
      merge_moments(rows, mean, m2, h[0], h[1], h[2]);
    }
    const double q0 = q[bh * kD + lane], q1 = q[bh * kD + 64 + lane];
    double qq = q0 * q0 + q1 * q1;
    for (int d = 1; d < 64; d <<= 1) {
      const double r2 = __shfl_xor(rows, d), mean2 = __shfl_xor(mean, d), m22 = __shfl_xor(m2, d);
      merge_moments(rows, mean, m2, r2, mean2, m22);
      qq += __shfl_xor(qq, d);
    }
    if (lane == 0) sigma2_hat[bh] = (cnt > 0 && qq > 0.0) ? (float)(m2 / (double)cnt / qq) : 0.f;
  }
}

// ----------------------------------------------------------------------------- launchers
// Workgroups that share a KV group in the two history kernels: two rounds of one workgroup per CU over all groups
// (lengths differ), but no more than one 128-row tile per wave needs.  One workgroup fills a CU's LDS and a tile is 128 rows,
// so time goes in steps of 2048 waves x 128 rows: 8 groups, tables from 32 queries in all, 101 to 104 us for 16K to 32768
// rows, 163 us for 33000, 187 to 201 us for 37K to 65K.
static int hist_blocks(const Shape& s) {
  const int groups = s.B * s.Hkv;
  const int most = (s.Lcap + kHistRows * kHistWaves - 1) / (kHistRows * kHistWaves);
  int n = 512 / groups;
  n = n < 1 ? 1 : n;
  return n < most ? n : most;
}

static int moment_chunks(const Shape& s) { return (s.Lcap + kMomentRows - 1) / kMomentRows; }

int64_t table_init_scratch_bytes(const Shape& s) {
  const int64_t stats = (int64_t)s.B * s.Hkv * hist_blocks(s) * kHistBatch * s.G * (8 + 4);
  const int64_t moments = (int64_t)s.B * s.Hq * moment_chunks(s) * 12 * 8;
  return stats + moments;
}

// Up to how many bytes of keys the pass over K above reads with ordinary loads.  With few queries it is bound by the bytes of K, and
// keys that will not be found in the memory-side cache again are read past it (one query, 64 groups x 32K rows, 537 MB: 119 -> 96
// us).  With one query the next reader is the next call, and the tables, written whole in between, take their part of the cache:
// tables of 4 x capacity, K + tables 224 MB 54.2 us kept, 58.4 past the caches, 280 MB 74.0 and 72.8, 336 MB 91.2 and 79.1.  With
// more queries k_hist_apply reads the keys again at once, while it writes the tables: 4 queries, keys + tables of 128 + 192 MB
// 135.9 and 153.1, 192 + 36 MB 120.7 and 122.4, 224 + 168 MB 164.6 and 163.3, 256 + 192 MB 199.3 and 186.2.  With 32 queries the
// matrix units bound the pass, and their operands leave no LDS for this form.
constexpr int kOnceQueries = 8;
static float stats_kept_bytes(const Shape& s, int n_queries) {
  const float tables = 12.f * s.B * s.Hq * s.Lcap;
  return n_queries == 1 ? (float)kKeptBytes - tables : 280.f * (1 << 20) - 0.5f * tables;
}

// Called once per context in table mode: the operands of 32 queries need more dynamic LDS than the default limit.
hipError_t configure_table_history(const Shape& s, int k_kind) {
  hipError_t e = hipSuccess;
  auto raise = [&](const void* kernel) {
    if (e == hipSuccess) e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, hist_lds(kHistBatch));
  };
#define LFPS_RAISE_HIST(GG, KIND)                                     \
  if (s.G == GG && k_kind == KIND) {                                  \
    raise((const void*)k_hist_stats<GG, false, KIND, false>);         \
    raise((const void*)k_hist_stats<GG, true, KIND, false>);          \
    raise((const void*)k_hist_stats<GG, false, KIND, true>);          \
    raise((const void*)k_hist_stats<GG, true, KIND, true>);           \
    raise((const void*)k_hist_apply<GG, false, KIND>);                \
    raise((const void*)k_hist_apply<GG, true, KIND>);                 \
  }
#define LFPS_RAISE_HIST_G(KIND) LFPS_RAISE_HIST(1, KIND) LFPS_RAISE_HIST(2, KIND) LFPS_RAISE_HIST(4, KIND)
  LFPS_RAISE_HIST_G(kKindBf16)
  LFPS_RAISE_HIST_G(kKindFp8)
  LFPS_RAISE_HIST_G(kKindF16)
#undef LFPS_RAISE_HIST_G
#undef LFPS_RAISE_HIST
  return e;
}

template <int G, bool kPaged, int kKind>
static hipError_t launch_hist_t(const Shape& s, float* tab_ver, float* tab_sla, const float* q0, int64_t q_stride,
                                int j0, int nq, int n_queries, double gamma, const KvView& kv, float* dots,
                                int64_t dots_stride, void* scratch, int32_t* flags, hipStream_t st) {
  const int bpg = hist_blocks(s), chunks = moment_chunks(s);
  double* moments = static_cast<double*>(scratch);
  double* part_l = moments + (int64_t)s.B * s.Hq * chunks * 12;
  float* part_m = reinterpret_cast<float*>(part_l + (int64_t)s.B * s.Hkv * bpg * kHistBatch * G);
  const dim3 grid(bpg, s.B * s.Hkv), block(kHistWaves * 64);
  const bool one = n_queries == 1;
  constexpr int kTurns = kHistWaves * StreamTile<kKind>::kLdsChunks * 16;
  static_assert(hist_lds(kOnceQueries) + kTurns <= hist_lds(kHistBatch), "the kernels' limit of dynamic LDS");
#define LFPS_STATS(ONCE, LDS)                                                                                          \
  hipLaunchKernelGGL((k_hist_stats<G, kPaged, kKind, ONCE>), grid, block, LDS, st, s, q0, q_stride, j0, nq, kv.k,      \
                     kv.stride_b, kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, part_m, part_l, one ? dots : nullptr, \
                     dots_stride, flags, kept)
  const float kept = stats_kept_bytes(s, n_queries);
  if (nq <= kOnceQueries && (float)s.B * s.Hkv * s.Lcap * (kD * KSub<kKind>::kElemBytes) > kept) LFPS_STATS(true, hist_lds(nq) + kTurns);
  else LFPS_STATS(false, hist_lds(nq));
#undef LFPS_STATS
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (one)
    hipLaunchKernelGGL(k_hist_apply_one, dim3(chunks, s.B * s.Hq), dim3(256), 0, st, s, tab_ver, tab_sla, dots,
                       dots_stride, kv.seq_lens, part_m, part_l, bpg, gamma, moments);
  else
    hipLaunchKernelGGL((k_hist_apply<G, kPaged, kKind>), grid, block, hist_lds(nq), st, s, tab_ver, tab_sla, q0, q_stride,
                       j0, nq, kv.k, kv.stride_b, kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, part_m, part_l, gamma,
                       n_queries);
  return hipGetLastError();
}

static hipError_t launch_hist(const Shape& s, float* tab_ver, float* tab_sla, const float* q0, int64_t q_stride, int j0,
                              int nq, int n_queries, double gamma, const KvView& kv, float* dots, int64_t dots_stride,
                              void* scratch, int32_t* flags, hipStream_t st) {
#define LFPS_HIST_ARGS s, tab_ver, tab_sla, q0, q_stride, j0, nq, n_queries, gamma, kv, dots, dots_stride, scratch, flags, st
#define LFPS_HIST(GG, KIND)                                                        \
  return kv.page.table ? launch_hist_t<GG, true, KIND>(LFPS_HIST_ARGS)             \
                       : launch_hist_t<GG, false, KIND>(LFPS_HIST_ARGS)
#define LFPS_HIST_G(KIND)                       \
  switch (s.G) {                                \
    case 1: LFPS_HIST(1, KIND);                 \
    case 2: LFPS_HIST(2, KIND);                 \
    case 4: LFPS_HIST(4, KIND);                 \
    default: return hipErrorInvalidValue;       \
  }
  if (kv.k_fp8) LFPS_HIST_G(kKindFp8)
  if (kv.f16) LFPS_HIST_G(kKindF16)
  LFPS_HIST_G(kKindBf16)
#undef LFPS_HIST_G
#undef LFPS_HIST
#undef LFPS_HIST_ARGS
}

hipError_t launch_table_history(const Shape& s, float* tab_ver, float* tab_sla, const float* q_hist, int n_queries,
                                double gamma, const KvView& kv, float* dots, int64_t dots_stride, void* scratch,
                                int32_t* flags, hipStream_t st) {
  const int64_t q_stride = (int64_t)s.B * s.Hq * kD;
  for (int j0 = 1; j0 <= n_queries; j0 += kHistBatch) {
    const int nq = n_queries - j0 + 1 < kHistBatch ? n_queries - j0 + 1 : kHistBatch;
    const hipError_t e = launch_hist(s, tab_ver, tab_sla, q_hist + (int64_t)(j0 - 1) * q_stride, q_stride, j0, nq,
                                     n_queries, gamma, kv, dots, dots_stride, scratch, flags, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_table_state(const Shape& s, const float* tab_ver, const float* tab_sla, double* state,
                              const int32_t* seq_lens, void* scratch, bool have_moments, hipStream_t st) {
  const int chunks = moment_chunks(s);
  double* part = static_cast<double*>(scratch);
  if (!have_moments)
    hipLaunchKernelGGL(k_table_moments, dim3(chunks, s.B * s.Hq), dim3(256), 0, st, s, tab_ver, tab_sla, seq_lens, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_table_state, dim3(s.B * s.Hq), dim3(192), 0, st, s, part, chunks, state, seq_lens);
  return hipGetLastError();
}

// The rows of a group are cut so that about 1024 workgroups share K and V, each with at least 256 rows, but into at least
// four parts: a lane then adds n / 64 rows in fp32 at most, however many groups there are (8192 rows with a mean of 0.5, RMS
// error of the mean: 1.7e-8; with one part for each of 1024 groups, n / 16 rows a lane, 3.9e-8).
static int prior_splits(const Shape& s) {
  const int by_len = (s.Lcap + 255) / 256;
  int n = (1024 + s.B * s.Hkv - 1) / (s.B * s.Hkv);
  n = n < by_len ? n : by_len;
  return n < 4 ? 4 : n;
}

int64_t prior_scratch_bytes(const Shape& s) {
  return (int64_t)s.B * s.Hkv * prior_splits(s) * prior_partial(s.G) * 8;
}

template <typename TK, typename T>
static hipError_t launch_priors_t(const Shape& s, const float* q, const KvView& kv, float* kbar, float* vbar,
                                  float* sigma2_hat, double* part, int32_t* flags, hipStream_t st) {
  const float scale = 0.08838834764831845f;
  const int splits = prior_splits(s);
  const dim3 grid(splits, s.B * s.Hkv), block(kPriorThreads);
#define LFPS_LAUNCH_PRI(GG, PAGED)                                                                                \
  hipLaunchKernelGGL((k_prior_partials<TK, T, GG, PAGED>), grid, block, 0, st, s, q, (const TK*)kv.k,             \
                     (const T*)kv.v, kv.stride_b, kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, part, scale, flags)
#define LFPS_LAUNCH_PRI_G(GG)                     \
  if (kv.page.table) LFPS_LAUNCH_PRI(GG, true);   \
  else LFPS_LAUNCH_PRI(GG, false)
  switch (s.G) {
    case 1: LFPS_LAUNCH_PRI_G(1); break;
    case 2: LFPS_LAUNCH_PRI_G(2); break;
    case 4: LFPS_LAUNCH_PRI_G(4); break;
    default: return hipErrorInvalidValue;
  }
#undef LFPS_LAUNCH_PRI_G
#undef LFPS_LAUNCH_PRI
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_prior_final, dim3(s.B * s.Hkv), dim3(1024), 0, st, s, q, kv.seq_lens, part, splits, kbar, vbar,
                     sigma2_hat);
  return hipGetLastError();
}

hipError_t launch_priors(const Shape& s, int dtype, const float* q, const KvView& kv, float* kbar, float* vbar,
                         float* sigma2_hat, void* scratch, int32_t* flags, hipStream_t st) {
  double* part = static_cast<double*>(scratch);
#define LFPS_PRI_ARGS s, q, kv, kbar, vbar, sigma2_hat, part, flags, st
  if (dtype == LFPS_BF16 && kv.k_fp8 && kv.v_fp8) return launch_priors_t<uint8_t, uint8_t>(LFPS_PRI_ARGS);
  if (dtype == LFPS_BF16 && kv.k_fp8) return launch_priors_t<uint8_t, uint16_t>(LFPS_PRI_ARGS);
  if (dtype == LFPS_BF16 && kv.v_fp8) return launch_priors_t<uint16_t, uint8_t>(LFPS_PRI_ARGS);
  if (dtype == LFPS_F16) return launch_priors_t<_Float16, _Float16>(LFPS_PRI_ARGS);
  if (dtype == LFPS_BF16) return launch_priors_t<uint16_t, uint16_t>(LFPS_PRI_ARGS);
  return launch_priors_t<float, float>(LFPS_PRI_ARGS);
#undef LFPS_PRI_ARGS
}

}  // namespace lfps
