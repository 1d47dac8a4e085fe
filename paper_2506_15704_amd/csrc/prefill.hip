// What prefill hands to decode: the score tables from the last s prefill queries (Eq. 4), their statistics, and the
// priors of the head-sparsity test (Sec. 4.2 "Prefilling", last paragraph).
//
// Eq. 4 needs, for every one of s queries and every head, the softmax of its scores over all rows it sees.  One query
// at a time that is s passes over K (16-bit keys at 8 groups x 32K rows: 14 us of scoring that writes every score, and
// 30 us of softmax and accumulation that reads and writes scores and tables, per query: 1.4 ms for s = 32).  K is the
// same for all of them, so 32 queries are taken together:
//   k_batch_stats   per (query, head) the largest score and the sum of exponentials, in one pass over K;
//   k_batch_apply   the scores once more (the same bits), the weights, and the sums over the queries, which never leave
//                   the chip: every table entry is written once.
// Two passes over K are needed because a weight needs the sum over all rows; storing the scores between them would
// cost 4 bytes per row, query and head (8.6 times the bytes of a second pass over bf16 keys at s = 32, G = 4).
// With many queries both are bound by the matrix and vector units: per 16 rows and 16 (query, head) pairs 12 products of 16
// cycles, of which a SIMD can issue two vector instructions each for nothing, and about 22 vector instructions in the first
// kernel, 45 in the second.  32 queries of 8 groups x 32K rows: 31 + 41 us (11 + 11 by the products alone), of 64 groups x 64K
// rows 331 + 453; before, one wave holding 128 rows and walking the queries, 49 + 59 and 1140 together.  With few queries they
// are bound by the bytes of K: 4 queries of 64 groups x 64K rows 157 + 265 us for 1.07 GB each and 0.2 GB of tables.
// A single query takes k_hist_stats and k_hist_apply_one instead: its scores are few enough to store.
#include "lfps_internal.h"
#include "score_mfma.h"

#include <float.h>

#include <type_traits>

namespace lfps {

constexpr int kHistWaves = 8;          // of a workgroup
constexpr int kHistSub = 8;            // 16-row sub-tiles a wave of k_hist_stats holds: 128 rows, which fill its registers
constexpr int kHistRows = 16 * kHistSub;
constexpr float kNoScore = -FLT_MAX;   // stands for "row not seen"
constexpr float kLeastMax = -1.7e38f;  // the largest score is taken as at least this: a row not seen weighs 0 beside any

// kHistSub sub-tiles of K rows as MFMA operands: lane (j, kb) holds its channels of the rows base + 16 t + j.  Rows past the
// sequence read its last row.
template <bool kPaged, int kKind>
struct HistTile {
  static constexpr int NT = kHistSub;
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
  // v[t] = q . K (not yet divided by sqrt(D)) of my row of sub-tile t for head kb
  __device__ __forceinline__ void dots(const Op (&A)[4], float (&v)[NT]) const {
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

// One query, which sees the offloaded rows [n_sink, n).  grid (blocks per group, B*Hkv).  part_m / part_l [bg, block, jq, h]
// (jq = 0): the largest q . K and the sum of the exponentials relative to it over the rows of the block (kLeastMax and 0 when it
// has none).  dots [B, Hq, stride]: every q . K.
// kMayOnce: rows past the caches (StreamTile) where the requests hold more than kept_bytes of them, see stats_kept_bytes.
template <int G, bool kPaged, int kKind, bool kMayOnce>
__global__ __launch_bounds__(kHistWaves * 64) void k_hist_stats(
    Shape s, const float* __restrict__ q, const void* __restrict__ K, int64_t stride_b, int64_t stride_h, int64_t stride_n,
    KvPage pg, const int32_t* __restrict__ seq_lens, float* __restrict__ part_m, double* __restrict__ part_l,
    float* __restrict__ dots, int64_t dots_stride, int32_t* __restrict__ flags, float kept_bytes) {
  request_arguments<decltype(&k_hist_stats<G, kPaged, kKind, kMayOnce>)>();
  using Tile = HistTile<kPaged, kKind>;
  using Op = typename Tile::Op;
  __shared__ u32x4 turn[kMayOnce ? kHistWaves : 1][StreamTile<kKind>::kLdsChunks];
  __shared__ float wm[kHistWaves][4];
  __shared__ double wl[kHistWaves][4];
  const int bg = blockIdx.y, b = bg / s.Hkv, g = bg % s.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, kb = lane >> 4;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const float held = kMayOnce ? held_rows(s, seq_lens) : 0.f;
  const int64_t head0 = (int64_t)b * s.Hq + (int64_t)g * G;
  // fp16: the query is split behind the requests for the first rows, beside their latency, as the compiler does by itself where there is
  // no range to report (8 groups x 32K rows 24.9 -> 23.8 us, x 128K 75.4 -> 72.9; of FP8 keys it takes 2.5 % longer).
  constexpr bool kSplitLate = Split3<Op>::kHalf;
  Op A[4] = {};
  QueryRows query;
  query.load(q, head0, G, j, kb);
  if constexpr (!kSplitLate) report_q_range(query.operand(A, G, j), flags);
  const bool once = kMayOnce && outgrow_cache(s, held, kD * KSub<kKind>::kElemBytes, kept_bytes);
  const char* Kbg = static_cast<const char*>(K) + RowMap<kPaged>::base(b, g, stride_b, stride_h) * KSub<kKind>::kElemBytes;
  float* my_dots = kb < G ? dots + (head0 + kb) * dots_stride : nullptr;
  float m = kLeastMax;                                     // of head kb (all sixteen lanes)
  double sum = 0.0;
  int lo, hi;
  wave_run((n + kHistRows - 1) / kHistRows, blockIdx.x * kHistWaves + wave, gridDim.x * kHistWaves, lo, hi);
  for (int tile = lo; tile < hi; ++tile) {
    const int base = tile * kHistRows;
    Tile T;
    if (kMayOnce && once)                                  // (a copy of the loop each: 1.5 us slower at 64 groups x 17K rows)
      T.load_once(Kbg, pg, b, stride_b, stride_n, base, n, lane, turn[kMayOnce ? wave : 0]);
    else
      T.load(Kbg, pg, b, stride_b, stride_n, base, n, j, kb);
    __builtin_amdgcn_sched_barrier(0);                     // (all rows asked for before the first product)
    if (kSplitLate && tile == lo) report_q_range(query.operand(A, G, j), flags);
    float v[kHistSub];
    T.dots(A, v);
    if (!(base >= s.n_sink && base + kHistRows <= n)) {    // (wave-uniform)
#pragma unroll
      for (int t = 0; t < kHistSub; ++t) {
        const int row = base + 16 * t + j;
        v[t] = row >= s.n_sink && row < n ? v[t] : kNoScore;
      }
    }
    float mx = v[0];
#pragma unroll
    for (int t = 1; t < kHistSub; ++t) mx = fmaxf(mx, v[t]);
    const float top = fmaxf(m, row16_max(mx));
    double l = 0.0;
#pragma unroll
    for (int t = 0; t < kHistSub; ++t) l += (double)exp_below<true>(v[t] - top);
    sum = sum * (double)exp_below<true>(m - top) + row16_sum(l);
    m = top;
    if (my_dots) {
#pragma unroll
      for (int t = 0; t < kHistSub; ++t) {
        const int row = base + 16 * t + j;
        if (row < n) my_dots[row] = v[t];
      }
    }
  }
  if (kSplitLate && n == 0) report_q_range(query.operand(A, G, j), flags);
  if (j == 0) {
    wm[wave][kb] = m;
    wl[wave][kb] = sum;
  }
  __syncthreads();
  if (tid < G) {
    float top = kLeastMax;
#pragma unroll
    for (int w = 0; w < kHistWaves; ++w) top = fmaxf(top, wm[w][tid]);
    double l = 0.0;
#pragma unroll
    for (int w = 0; w < kHistWaves; ++w) l += wl[w][tid] * (double)exp_below<true>(wm[w][tid] - top);
    const int64_t o = ((int64_t)bg * gridDim.x + blockIdx.x) * (kHistBatch * G) + tid;
    part_m[o] = top;
    part_l[o] = l;
  }
}

// The partials of one (query, head), merged by kPer neighbouring lanes (sub = 0 .. kPer - 1): the largest dot
// product, and the factor 1 / (2 s (1 - gamma) sum) that turns an exponential into a table contribution.  weight(x): the
// exponential of a difference x of two of the partials' maxima.
template <int kPer, typename Weight>
__device__ __forceinline__ void merge_hist(const float* part_m, const double* part_l, int64_t o, int64_t step, int blocks,
                                           int sub, double gamma, int n_queries, float& m, double& norm, Weight weight) {
  m = kLeastMax;
  double l = 0.0;
  if constexpr (kPer > 4) {
#pragma unroll 8
    for (int k = sub; k < blocks; k += kPer) m = fmaxf(m, part_m[o + k * step]);
#pragma unroll
    for (int d = 1; d < kPer; d <<= 1) m = fmaxf(m, __shfl_xor(m, d));
#pragma unroll 8
    for (int k = sub; k < blocks; k += kPer) l += part_l[o + k * step] * (double)weight(part_m[o + k * step] - m);
  } else {
    // Eight loads of a lane at a time, also of the last ones (one by one, up to seven of them in turn: 8 queries of 8 groups x 3600 FP8
    // rows 20.6 us instead of 16.9).  The conditions on first are the same for all lanes; past the end a lane reads partial 0 and counts
    // nothing.
    constexpr int kAtOnce = 8;
    auto batches = [&](auto batch) {
      int first = 0;
      for (; first + kAtOnce * kPer <= blocks; first += kAtOnce * kPer) batch(std::true_type{}, first);
      if (first < blocks) batch(std::false_type{}, first);
    };
    batches([&](auto whole, int first) __attribute__((always_inline)) {
      constexpr bool kWhole = decltype(whole)::value;
      float x[kAtOnce];
#pragma unroll
      for (int u = 0; u < kAtOnce; ++u) {
        const int k = first + u * kPer + sub;
        x[u] = kLeastMax;
        if (kWhole || first + u * kPer < blocks) x[u] = part_m[o + (kWhole || k < blocks ? k : 0) * step];
      }
#pragma unroll
      for (int u = 0; u < kAtOnce; ++u) m = fmaxf(m, x[u]);
    });
#pragma unroll
    for (int d = 1; d < kPer; d <<= 1) m = fmaxf(m, __shfl_xor(m, d));
    batches([&](auto whole, int first) __attribute__((always_inline)) {
      constexpr bool kWhole = decltype(whole)::value;
      float x[kAtOnce];
      double part[kAtOnce];
#pragma unroll
      for (int u = 0; u < kAtOnce; ++u) {
        const int k = first + u * kPer + sub;
        x[u] = kLeastMax;
        part[u] = 0.0;
        if (kWhole || first + u * kPer < blocks) {
          const int64_t at = o + (kWhole || k < blocks ? k : 0) * step;
          x[u] = part_m[at];
          part[u] = part_l[at];
        }
      }
#pragma unroll
      for (int u = 0; u < kAtOnce; ++u)
        if (kWhole || first + u * kPer < blocks)
          l += kWhole || first + u * kPer + sub < blocks ? part[u] * (double)weight(x[u] - m) : 0.0;
    });
  }
#pragma unroll
  for (int d = 1; d < kPer; d <<= 1) l += __shfl_xor(l, d);
  norm = l > 0.0 ? 1.0 / (2.0 * (double)n_queries * (1.0 - gamma) * l) : 0.0;
}

// e * norm rounded once to fp32 (norm = hi + lo).
__device__ __forceinline__ float weigh(float e, float hi, float lo) { return fmaf(e, hi, e * lo); }

// M1..M4 of a table's entries, then the smallest and the negated largest.
struct TableMoments {
  double m[4] = {0, 0, 0, 0};
  float e[2] = {INFINITY, INFINITY};
  __device__ __forceinline__ void add(float x) {
    const double a = x;
    m[0] += a; m[1] += a * a; m[2] += a * a * a; m[3] += a * a * a * a;
    e[0] = fminf(e[0], x); e[1] = fminf(e[1], -x);
  }
  __device__ __forceinline__ void reduce_wave() {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      m[p] = row16_sum(m[p]);
      m[p] += __shfl_xor(m[p], 16);
      m[p] += __shfl_xor(m[p], 32);
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      e[p] = -row16_max(-e[p]);
      e[p] = fminf(e[p], __shfl_xor(e[p], 16));
      e[p] = fminf(e[p], __shfl_xor(e[p], 32));
    }
  }
  __device__ __forceinline__ void store(double* to) const {                // six values
#pragma unroll
    for (int p = 0; p < 4; ++p) to[p] = m[p];
#pragma unroll
    for (int p = 0; p < 2; ++p) to[4 + p] = (double)e[p];
  }
};

// Of both tables' entries of a workgroup (256 threads, U positions each, those with in[u]): M1..M4 of the vertical and of the slash
// table, then the smallest and the negated largest of both, to out[0:12].
template <int U>
__device__ __forceinline__ void moments_of_chunk(const float (&xv)[U], const float (&xs)[U], const bool (&in)[U],
                                                 double* __restrict__ out) {
  __shared__ double red[4][2][6];
  const int tid = threadIdx.x;
  TableMoments v, x;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (!in[u]) continue;
    v.add(xv[u]);
    x.add(xs[u]);
  }
  v.reduce_wave();
  x.reduce_wave();
  if ((tid & 63) == 0) {
    v.store(red[tid >> 6][0]);
    x.store(red[tid >> 6][1]);
  }
  __syncthreads();
  if (tid < 12) {
    const int table = tid < 8 ? tid >> 2 : (tid - 8) >> 1, at = tid < 8 ? tid & 3 : 4 + (tid & 1);
    double t = red[0][table][at];
    for (int w = 1; w < 4; ++w) t = tid < 8 ? t + red[w][table][at] : fmin(t, red[w][table][at]);
    out[tid] = t;
  }
}

// ----------------------------------------------------------------------------- many queries
// Both kernels take the K rows of a workgroup in chunks through LDS (as 16-bit operands, two chunks there and one
// more on its way in registers), and every wave keeps its queries: sixteen (query, head) pairs, a unit, are the sixteen rows
// of an MFMA A operand, the three terms of the query one operand each.  (With the terms as rows of one operand, sixteen rows were
// four heads of one query and four of them zeros; with the rows in registers and the queries walked, every workgroup first
// loaded all of its rows and then computed, and each query's maximum and sum took a reduction over lanes per 128 rows.)
// U waves (1, 2, 4, 8) of the eight of a workgroup hold the units of a batch; where that is not all eight, the workgroup's rows are
// cut into 8 / U spans of their own, and a chunk of R rows holds R U / 8 of each.  Row 4 i + c of an operand (D: lane group i,
// register c) is query 4 quad + c, quad = unit * 4 / G + i / G, of head i % G.
constexpr int kBatchThreads = 64 * kHistWaves;
// 16-byte pieces from row to row, and the piece that lane group kb takes at step kk: a read of the wave is served 16 lanes at a
// time, lanes 0-3 and 12-15 of an even group with 4-11 of the next odd one and the other way round, which meet in no bank so (with
// rows 17 apart and pieces kk + 4 kb every read waited half its time again).
constexpr int kChunkPitch = kD / 8 + 2;
__device__ __forceinline__ constexpr int chunk_piece(int kk, int kb) { return 2 * kk + (kb & 1) + 8 * (kb >> 1); }
template <int U, int R>
struct BatchShape {
  static constexpr int kRows = R;
  static constexpr int kPieces = R * kChunkPitch;
  static constexpr int kSpans = kHistWaves / U;
  static constexpr int kSpanRows = R / kSpans;             // of a chunk
  static constexpr int kSubs = kSpanRows / 16;             // sub-tiles of 16 rows a wave takes of a chunk
};
constexpr int kApplyRows = 128;
// Rows of a chunk in the first kernel: 128 where a wave's span would be less than sixteen (one unit), and of FP8 keys where the
// registers of a wave allow it, 64 being few bytes on their way: 2 queries of one group (four heads) x 128K rows 32.9 -> 30.9 us, of
// 8 groups x 32K 34.6 -> 32.6, of 128 x 32K 274 -> 260, 16 of 64 x 16000 with two heads each 92.1 -> 86.1.
constexpr int stats_form(int U, int kind) {
  return U <= 2 && kind == kKindFp8 ? kPartsFp8 : (U == 1 ? kPartsOneUnit : kPartsShort);
}
constexpr int stats_rows(int form) { return form == kPartsShort ? 64 : 128; }

// The rows of a workgroup's chunks: from memory to registers, from there to LDS, by the first kThreads of its threads.
template <bool kPaged, int kKind, typename B, int kThreads>
struct ChunkRows {
  static constexpr int kPieces = kD * KSub<kKind>::kElemBytes / 16;      // of a row
  static constexpr int kStep = kThreads / kPieces;                       // rows of one load
  static constexpr int kLoads = B::kRows / kStep;
  static_assert(kLoads * kStep == B::kRows, "whole loads");
  using Rows = RowMap<kPaged>;
  u32x4 raw[kLoads];
  int block[kPaged ? kLoads : 1];                          // paged: of my rows of the chunk to fetch next
  int next, span_rows, n;                                  // that chunk's first row, rows from span to span
  __device__ __forceinline__ int row_of(int i) const {     // (outside the sequence: a row of it)
    const int at = (int)threadIdx.x / kPieces + i * kStep;
    const int row = next + at / B::kSpanRows * span_rows + at % B::kSpanRows;
    return row < 0 ? 0 : (row < n ? row : n - 1);
  }
  __device__ __forceinline__ void look_up(const KvPage& pg, int b) {
    if constexpr (kPaged) {
#pragma unroll
      for (int i = 0; i < kLoads; ++i) block[i] = Rows::block(pg, b, row_of(i));
    }
  }
  __device__ __forceinline__ void start(const KvPage& pg, int b, int first, int span_rows_, int n_) {
    n = n_;
    next = first;
    span_rows = span_rows_;
    look_up(pg, b);
  }
  // my pieces of the next chunk; the block table is asked one chunk ahead.  (Its entries are used as they come only then: with the
  // physical rows kept instead, each look-up was waited for, and the rows asked for before it.  2 queries, pages of 64: 128 groups x
  // 32K FP8 rows 409 -> 273 us, contiguous 264; 64 x 16000 97.3 -> 81.9 and of bf16 111.4 -> 101.5, contiguous 74.6 and 96.7.)
  __device__ __forceinline__ void fetch(const char* Kbg, const KvPage& pg, int b, int64_t stride_b, int64_t stride_n, bool once) {
    auto at = [&](int i) {
      const int64_t o = Rows::offset_in(pg, block[kPaged ? i : 0], row_of(i), stride_b, stride_n);
      return reinterpret_cast<const u32x4*>(Kbg + o * KSub<kKind>::kElemBytes) + (int)threadIdx.x % kPieces;
    };
    if (once) {
      asm volatile("; past the caches");                   // (or the compiler makes ordinary loads of both branches)
#pragma unroll
      for (int i = 0; i < kLoads; ++i) raw[i] = __builtin_nontemporal_load(at(i));
      asm volatile("; past the caches");
    } else {
#pragma unroll
      for (int i = 0; i < kLoads; ++i) raw[i] = *at(i);
    }
    next += B::kSpanRows;
    look_up(pg, b);
  }
  __device__ __forceinline__ void put(u32x4* chunk) const {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      u32x4* to = chunk + ((int)threadIdx.x / kPieces + i * kStep) * kChunkPitch;
      if constexpr (kKind == kKindFp8) {
        to += 2 * ((int)threadIdx.x % kPieces);
        to[0] = __builtin_bit_cast(u32x4, fp8x8_to_bf16x8(raw[i][0], raw[i][1]));
        to[1] = __builtin_bit_cast(u32x4, fp8x8_to_bf16x8(raw[i][2], raw[i][3]));
      } else {
        to[(int)threadIdx.x % kPieces] = raw[i];
      }
    }
  }
};

// The A operands of a unit: the terms of 4 log2(e) / sqrt(D) times the queries, so that a quarter of a product is the power of two
// that its row weighs.  The factor is applied to more than 24 bits and the three terms hold that: a weight is then one fused
// subtraction of the maximum and one exp2, without the product of a rounded score with a rounded factor in between (with the
// plain queries, the factor and its rounding made good in exp_below, the vector instructions bound both kernels: 14 a product in
// the first and 17 in the second, now 6 and 11).  (4: an element of the largest size does not overflow.)
constexpr float kProductUnit = 0.25f;
__device__ __forceinline__ float product_weight(float x, float top) {
  return __builtin_amdgcn_exp2f(fmaf(x, kProductUnit, -kProductUnit * top));
}
template <int G, typename Op>
struct UnitQueries {
  Op a[3][4];
  __device__ static __forceinline__ void terms(float f, Op (&e)[3], int c) {
    constexpr double factor = 4.0 * 0.08838834764831845 * 1.4426950408889634;
    constexpr float hi = (float)factor, lo = (float)(factor - (double)hi);
    using Elem = std::remove_reference_t<decltype(e[0][0] + e[0][0])>;
    constexpr float kUp = Split3<Op>::kHalf ? 2048.0f : 1.0f;              // as Split3's terms are scaled
    float x = f * hi;
    asm("" : "+v"(x));                                     // (one value: not rounded to 16 bits from the product in one place)
    const float rest = fmaf(f, lo, fmaf(f, hi, -x));
    const Elem t0 = (Elem)x;
    x -= (float)t0;
    const Elem t1 = (Elem)(x * kUp);
    x = fmaf((float)t1, -1.0f / kUp, x) + rest;
    e[0][c] = t0;
    e[1][c] = t1;
    e[2][c] = (Elem)(x * (kUp * kUp));
  }
  // Returns true if it met an element beyond the fp16 range.
  __device__ __forceinline__ bool load(const float* __restrict__ q0, int64_t q_stride, int64_t head0, int nq, int unit, int lane) {
    const int m = lane & 15, i = m >> 2;
    const int jq = 4 * (unit * (4 / G) + i / G) + (m & 3);
    const bool live = jq < nq;
    const float4* p = reinterpret_cast<const float4*>(q0 + (live ? jq : 0) * q_stride + (head0 + i % G) * kD);
    float4 x[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) x[c] = p[2 * chunk_piece(c >> 1, lane >> 4) + (c & 1)];
    bool clipped = false;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const float4 lo = x[2 * kk], hi = x[2 * kk + 1];
      float f[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      if constexpr (Split3<Op>::kHalf) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          if (fabsf(f[c]) > 65504.0f) {
            clipped |= live;
            f[c] = copysignf(65504.0f, f[c]);
          }
        }
      }
      Op term[3];
#pragma unroll
      for (int c = 0; c < 8; ++c) terms(f[c], term, c);
      const uint32_t keep = live ? ~0u : 0u;
#pragma unroll
      for (int t = 0; t < 3; ++t) a[t][kk] = __builtin_bit_cast(Op, __builtin_bit_cast(u32x4, term[t]) & keep);
    }
    return clipped;
  }
  // [c]: the product of the unit's rows 4 (lane >> 4) + c with the K row of my lane & 15, whose operands are k.  bf16: all terms in
  // one sum, the small ones first.
  __device__ __forceinline__ f32x4 dots(const Op (&k)[4]) const {
    f32x4 acc[3] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    constexpr bool kApart = Split3<Op>::kHalf;             // fp16 terms are scaled differently
#pragma unroll
    for (int t = 2; t >= 0; --t)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) acc[kApart ? t : 0] = mfma16(a[t][kk], k[kk], acc[kApart ? t : 0]);
    if constexpr (kApart) {
      f32x4 v;
#pragma unroll
      for (int c = 0; c < 4; ++c)                          // (small ones first: the least of them alone would round away)
        v[c] = fmaf(fmaf(acc[2][c], 1.0f / 2048.0f, acc[1][c]), 1.0f / 2048.0f, acc[0][c]);
      return v;
    }
    return acc[0];
  }
};

// The operands of a K row in a chunk (x: the first piece of my lane group).
template <typename Op>
__device__ __forceinline__ void read_operands(Op (&k)[4], const u32x4* x) {
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) k[kk] = __builtin_bit_cast(Op, x[chunk_piece(kk, 0)]);
}

// The products of a wave's unit with the sub-tiles kFrom .. kSubs - 1 of a chunk (x: the first piece of my row of its first
// sub-tile), and beside those of a sub-tile what is to be done with the ones before: use(sub-tile, products), about kBeside vector
// instructions between two products.  (The matrix unit works on while a wave issues other instructions, two for each product; left
// to itself the compiler puts all products of a sub-tile first.)
template <int kSubs, int kFrom, int kBeside, int kAt, int G, typename Op, typename Use>
__device__ __forceinline__ void walk_chunk_from(const UnitQueries<G, Op>& queries, const u32x4* x, const Op (&k)[4], const f32x4& before,
                                                Use use) {
  Op ahead[4];
  if constexpr (kAt + 1 < kSubs) read_operands(ahead, x + 16 * (kAt + 1) * kChunkPitch);
  f32x4 v = before;
  if constexpr (kAt < kSubs) v = queries.dots(k);
  if constexpr (kAt > kFrom) use(kAt - 1, before);
  if constexpr (kAt > kFrom && kAt < kSubs) {
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);     // LDS reads
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);     // a product
      __builtin_amdgcn_sched_group_barrier(0x2, kBeside, 0);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (kAt < kSubs) walk_chunk_from<kSubs, kFrom, kBeside, kAt + 1>(queries, x, ahead, v, use);
}
template <int kSubs, int kFrom, int kBeside, int G, typename Op, typename Use>
__device__ __forceinline__ void walk_chunk(const UnitQueries<G, Op>& queries, const u32x4* x, Use use) {
  Op k[4];
  read_operands(k, x + 16 * kFrom * kChunkPitch);
  walk_chunk_from<kSubs, kFrom, kBeside, kFrom>(queries, x, k, f32x4{0.f, 0.f, 0.f, 0.f}, use);
}

// Where a workgroup and a wave of it work: chunks, and the rows [first, first + span_rows) of the wave's span.
template <int U, typename B>
struct BatchWork {
  int chunks, wg_first, wg_rows, unit, span, span_rows, first;
  __device__ __forceinline__ BatchWork(int n, int wave) {
    const int tiles = (n + B::kRows - 1) / B::kRows;
    const int per = (tiles + (int)gridDim.x - 1) / (int)gridDim.x;
    wg_rows = per * B::kRows;
    wg_first = (int)blockIdx.x * wg_rows;
    chunks = wg_first < n ? per : 0;                       // (workgroup-uniform)
    unit = wave % U;
    span = wave / U;
    span_rows = per * B::kSpanRows;
    first = wg_first + span * span_rows;
  }
};

// How far query jq of a batch of nq sees: rows below (0: no such query), and how far all queries of a unit that there are do.
__device__ __forceinline__ int seen_by(int jq, int j0, int nq, int n) { return jq < nq ? n - (j0 + jq) + 1 : 0; }
template <int G>
__device__ __forceinline__ int seen_by_all(int unit, int j0, int nq, int n) {
  const int last = (unit + 1) * (16 / G) - 1;
  return seen_by(last < nq ? last : nq - 1, j0, nq, n);
}

// grid (blocks per group, B*Hkv).  Queries j0 .. j0 + nq - 1 (j = 1: the most recent); query j sees the offloaded rows
// [n_sink, n - j + 1).  part_m / part_l [bg, block, jq, h]: the largest product and the sum of the weights relative to it over
// the rows of the block (kLeastMax and 0 when it has none).
// A lane keeps the maximum and the sum of its own rows (of four queries) to the end.  Two workgroups per CU: four waves on a SIMD,
// of which some are at their products while others are not.
template <int G, bool kPaged, int kKind, int U>
__global__ __launch_bounds__(kBatchThreads, 4) void k_batch_stats(
    Shape s, const float* __restrict__ q0, int64_t q_stride, int j0, int nq, const void* __restrict__ K,
    int64_t stride_b, int64_t stride_h, int64_t stride_n, KvPage pg, const int32_t* __restrict__ seq_lens,
    float* __restrict__ part_m, double* __restrict__ part_l, int32_t* __restrict__ flags, float kept_bytes) {
  using B = BatchShape<U, stats_rows(stats_form(U, kKind))>;
  using Op = typename KSub<kKind>::Operand;
  __shared__ u32x4 chunk[2][B::kPieces];
  __shared__ float wm[kHistWaves][16];
  __shared__ double wl[kHistWaves][16];
  const int bg = blockIdx.y, b = bg / s.Hkv, g = bg % s.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, kb = lane >> 4;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const bool once = outgrow_cache(s, held_rows(s, seq_lens), kD * KSub<kKind>::kElemBytes, kept_bytes);
  const BatchWork<U, B> work(n, wave);
  const char* Kbg = static_cast<const char*>(K) + RowMap<kPaged>::base(b, g, stride_b, stride_h) * KSub<kKind>::kElemBytes;
  float m[4];
  double l[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    m[c] = kLeastMax;
    l[c] = 0.0;
  }
  if (work.chunks > 0) {
    ChunkRows<kPaged, kKind, B, kBatchThreads> rows;
    rows.start(pg, b, work.wg_first, work.span_rows, n);
    rows.fetch(Kbg, pg, b, stride_b, stride_n, once);
    UnitQueries<G, Op> queries;
    report_q_range(queries.load(q0, q_stride, (int64_t)b * s.Hq + (int64_t)g * G, nq, work.unit, lane), flags);
    const int all_see = seen_by_all<G>(work.unit, j0, nq, n);
    const bool idle = work.unit * (16 / G) >= nq;          // (wave-uniform: a unit of no query)
    for (int at = 0; at < work.chunks; ++at) {
      rows.put(chunk[at & 1]);
      rows.fetch(Kbg, pg, b, stride_b, stride_n, once);
      __syncthreads();
      if (idle) continue;
      const u32x4* mine = chunk[at & 1] + (work.span * B::kSpanRows + j) * kChunkPitch + chunk_piece(0, kb);
      f32x4 x[B::kSubs];
#pragma unroll
      for (int t = 0; t < B::kSubs; ++t) {
        Op k[4];
        read_operands(k, mine + 16 * t * kChunkPitch);
        x[t] = queries.dots(k);
      }
      const int base = work.first + at * B::kSpanRows;
      if (!(base >= s.n_sink && base + B::kSpanRows <= all_see)) {         // (wave-uniform)
        const int jq = 4 * (work.unit * (4 / G) + kb / G);
#pragma unroll
        for (int t = 0; t < B::kSubs; ++t)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const int row = base + 16 * t + j;
            x[t][c] = row >= s.n_sink && row < seen_by(jq + c, j0, nq, n) ? x[t][c] : kNoScore;
          }
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float top = m[c];
#pragma unroll
        for (int t = 0; t < B::kSubs; ++t) top = __builtin_elementwise_maximum(top, x[t][c]);   // (a NaN is in the sum then, too)
        l[c] *= (double)product_weight(m[c], top);
        m[c] = top;
#pragma unroll
        for (int t = 0; t < B::kSubs; ++t) l[c] += (double)product_weight(x[t][c], top);
      }
    }
  }
  // the sixteen lanes of a row of lanes, then the spans
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float top = row16_max(m[c]);
    const double sum = row16_sum(l[c] * (double)product_weight(m[c], top));
    if (j == 0) {
      wm[wave][4 * kb + c] = top;
      wl[wave][4 * kb + c] = sum;
    }
  }
  __syncthreads();
  for (int e = tid; e < nq * G; e += kBatchThreads) {
    const int jq = e / G, h = e % G, quad = jq >> 2;
    const int unit = quad / (4 / G), at = 4 * (quad % (4 / G) * G + h) + (jq & 3);
    float top = kLeastMax;
#pragma unroll
    for (int w = 0; w < B::kSpans; ++w) top = fmaxf(top, wm[unit + U * w][at]);
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < B::kSpans; ++w) sum += wl[unit + U * w][at] * (double)product_weight(wm[unit + U * w][at], top);
    const int64_t o = ((int64_t)bg * gridDim.x + blockIdx.x) * (kHistBatch * G) + e;
    part_m[o] = top;
    part_l[o] = sum;
  }
}

// The same grid and queries.  Adds  w_j(i) / (2 s (1 - gamma))  to the vertical table at i and to the slash table at
// i + j - 1, for all nq queries at once; the first batch (j0 = 1) writes the tables whole (zeros past the sequence and
// in the lower half of the slash frame), later batches add to them.
// A lane has the weights of four queries of a quad for its row: their sum, and the sum in which each query's weight is moved
// one row up for every query before it in the quad (a rotation inside 16 lanes; what enters at the first row of sixteen comes
// from the sixteen before), go to LDS per quad and head, the latter four rows further up for every quad before.  One thread per
// row and head adds the quads up, a chunk behind the products.  A span starts with the 32 rows before it, for what reaches into
// it (31 rows at most).
// moments (or NULL; the only batch): the statistics of the workgroup's rows, as k_table_moments leaves them, one partial per
// workgroup.
template <int U>
struct ApplyLds {
  using B = BatchShape<U, kApplyRows>;
  static constexpr int kQuads = 4 * U;                     // times heads
  u32x4 chunk[2][B::kPieces];
  float sum[2][kQuads][B::kRows];                          // [quad * G + head][row of the chunk, span by span]
  float moved[B::kSpans][kQuads][3 * B::kSpanRows];        // per span, [row of three chunks in turn]
  float ref[3][4][kHistBatch];                             // [largest product, factor as a pair of floats][head][query]
};
template <int G, bool kPaged, int kKind, int U>
__global__ __launch_bounds__(kBatchThreads, 2) void k_batch_apply(
    Shape s, float* __restrict__ tab_ver, float* __restrict__ tab_sla, const float* __restrict__ q0, int64_t q_stride,
    int j0, int nq, const void* __restrict__ K, int64_t stride_b, int64_t stride_h, int64_t stride_n, KvPage pg,
    const int32_t* __restrict__ seq_lens, const float* __restrict__ part_m, const double* __restrict__ part_l,
    int parts, double gamma, int n_queries, double* __restrict__ moments) {
  using B = BatchShape<U, kApplyRows>;
  using Op = typename KSub<kKind>::Operand;
  using Lds = ApplyLds<U>;
  constexpr int kSpanRows = B::kSpanRows, kRing = 3 * kSpanRows;
  constexpr int kMostQuads = 4 * U / G;
  static_assert(4 * (kMostQuads - 1) + 15 < 2 * kSpanRows, "what is moved up ends in the next chunk");
  static_assert(4 * kMostQuads <= (kSpanRows < 32 ? kSpanRows : 32), "what reaches into a span comes from the rows before it that are taken");
  extern __shared__ char lds_raw[];
  Lds& lds = *reinterpret_cast<Lds*>(lds_raw);
  const int bg = blockIdx.y, b = bg / s.Hkv, g = bg % s.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, kb = lane >> 4;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const BatchWork<U, B> work(n, wave);
  const char* Kbg = static_cast<const char*>(K) + RowMap<kPaged>::base(b, g, stride_b, stride_h) * KSub<kKind>::kElemBytes;
  const int64_t head0 = (int64_t)b * s.Hq + (int64_t)g * G;
  const bool first = j0 == 1;
  // The first four waves fetch the rows, the others add up and write the tables: a wait for a load would wait for the stores
  // before it.  What a wave of the latter adds up: the rows of a chunk, of one head.
  constexpr int kLoadThreads = kBatchThreads / 2;
  const int my_head = wave - kHistWaves / 2;
  TableMoments stats_v, stats_s;
  if (work.chunks > 0) {
    UnitQueries<G, Op> queries;                            // (k_batch_stats reported the range)
    (void)queries.load(q0, q_stride, head0, nq, work.unit, lane);
    {
      static_assert(kBatchThreads == kHistBatch * 4 * 4, "four lanes per query and head");
      const int jq = tid >> 4, h = (tid >> 2) & 3, sub = tid & 3;
      float top = 0.f;
      double norm = 0.0;
      if (jq < nq && h < G)                                // uniform over the four lanes
        merge_hist<4>(part_m, part_l, (int64_t)bg * parts * (kHistBatch * G) + jq * G + h, kHistBatch * G, parts,
                      sub, gamma, n_queries, top, norm, [](float x) { return product_weight(x, 0.f); });
      const float hi = (float)norm;
      lds.ref[0][h][jq] = top;
      lds.ref[1][h][jq] = hi;
      lds.ref[2][h][jq] = (float)(norm - (double)hi);
    }
    const bool idle = work.unit * (16 / G) >= nq;          // (wave-uniform: a unit of no query)
    const int quads = (nq + 3) >> 2;
    const int all_see = seen_by_all<G>(work.unit, j0, nq, n);
    const int quad = work.unit * (4 / G) + kb / G;
    const float* my_ref = &lds.ref[0][kb % G][(4 * quad) & (kHistBatch - 1)];
    float enter[3] = {0.f, 0.f, 0.f};                      // the rotated sums of the sixteen rows before
    // masked 0: every row is seen by all queries of the unit, 1: by those that there are, 2: a row may not be seen.  (A query that is
    // not there has to be left out: its products are zeros, but not with a row that is not finite.)
    constexpr std::integral_constant<int, 0> kFull{};
    constexpr std::integral_constant<int, 1> kPart{};
    constexpr std::integral_constant<int, 2> kRows{};
    const bool full = (work.unit + 1) * (16 / G) <= nq;    // (wave-uniform)
    auto products = [&](auto from, auto masked, const u32x4* buf, int at, int sum_at, int moved_at) __attribute__((always_inline)) {
      constexpr int kMasked = decltype(masked)::value;
      const int row0 = work.first + at * kSpanRows + j;
      const u32x4* mine = buf + (work.span * kSpanRows + j) * kChunkPitch + chunk_piece(0, kb);
      float* sum = &lds.sum[sum_at][work.unit * 4 + kb][work.span * kSpanRows + j];
      float* moved = lds.moved[work.span][work.unit * 4 + kb];
      const f32x4 top = *reinterpret_cast<const f32x4*>(my_ref), hi = *reinterpret_cast<const f32x4*>(my_ref + 4 * kHistBatch),
                  lo = *reinterpret_cast<const f32x4*>(my_ref + 8 * kHistBatch);
      walk_chunk<B::kSubs, decltype(from)::value, kMasked == 2 ? 5 : 3>(queries, mine, [&](int t, const f32x4& v) __attribute__((always_inline)) {
        float w[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          float x = v[c];
          if constexpr (kMasked == 2)
            x = row0 + 16 * t >= s.n_sink && row0 + 16 * t < seen_by(4 * quad + c, j0, nq, n) ? x : kNoScore;
          w[c] = weigh(product_weight(x, top[c]), hi[c], lo[c]);
          if constexpr (kMasked == 1) w[c] = 4 * quad + c < nq ? w[c] : 0.f;
        }
        float up = w[3];
#pragma unroll
        for (int c = 2; c >= 0; --c) {
          const float r = row16_rotate<1>(up);
          up = (j != 0 ? r : enter[c]) + w[c];
          enter[c] = r;
        }
        sum[16 * t] = ((w[3] + w[2]) + w[1]) + w[0];
        int to = moved_at * kSpanRows + 16 * t + 4 * quad + j;
        if (t + 2 >= B::kSubs) to = to < kRing ? to : to - kRing;
        moved[to] = up;
      });
    };
    // the quads of a chunk, by one thread per row and head
    auto combine = [&](int at, int sum_at, int moved_at) __attribute__((always_inline)) {
      if (my_head >= G) return;
      float* ver = tab_ver + (head0 + my_head) * s.Lcap;
      float* sla = tab_sla + (head0 + my_head) * 2 * s.Lcap;               // position p of an untouched table is slot Lcap + p
#pragma unroll
      for (int i = 0; i < B::kRows / 64; ++i) {
        const int my_at = 64 * i + lane, my_span = my_at / kSpanRows, my_row = my_at % kSpanRows;
        const float* sum = &lds.sum[sum_at][my_head][my_at];
        const float* moved = &lds.moved[my_span][my_head][moved_at * kSpanRows + my_row];
        float av = 0.f, as = 0.f;
#pragma unroll
        for (int quad = Lds::kQuads / G - 1; quad >= 0; --quad) {          // (all reads at once: no branch at a quad that is not there)
          const float v = sum[quad * G * B::kRows], x = moved[quad * G * kRing];
          av += quad < quads ? v : 0.f;
          as += quad < quads ? x : 0.f;
        }
        const int row = work.wg_first + my_span * work.span_rows + at * kSpanRows + my_row, pos = row + j0 - 1;
        if (first) {
          if (row < s.Lcap) {                              // past the sequence the sums are zero
            ver[row] = av;
            sla[s.Lcap + row] = as;
            sla[row] = 0.f;
            if (moments && row >= s.n_sink && row < n) {
              stats_v.add(av);
              stats_s.add(as);
            }
          }
        } else {
          if (row < n) ver[row] += av;
          if (pos < n) sla[s.Lcap + pos] += as;
        }
      }
    };
    const bool loads = wave < kHistWaves / 2;              // (wave-uniform; the barriers stand outside of what it decides)
    ChunkRows<kPaged, kKind, B, kLoadThreads> rows;
    if (loads) {
      rows.start(pg, b, work.wg_first - kSpanRows, work.span_rows, n);     // chunk -1: the rows before the spans
      rows.fetch(Kbg, pg, b, stride_b, stride_n, false);
      rows.put(lds.chunk[1]);
      rows.fetch(Kbg, pg, b, stride_b, stride_n, false);
    }
    __syncthreads();
    constexpr std::integral_constant<int, 0> kWhole{};
    constexpr std::integral_constant<int, (B::kSubs > 2 ? B::kSubs - 2 : 0)> kLast{};      // the last 32 rows
    if (!idle) products(kLast, kRows, lds.chunk[1], -1, 1, 2);
    int moved_at = 0;                                      // chunk at % 3
    for (int at = 0; at < work.chunks; ++at) {
      if (loads) {
        rows.put(lds.chunk[at & 1]);
        rows.fetch(Kbg, pg, b, stride_b, stride_n, false);
      }
      __syncthreads();
      if (!loads && at > 0) combine(at - 1, (at - 1) & 1, moved_at > 0 ? moved_at - 1 : 2);
      const int base = work.first + at * kSpanRows;
      if (idle) {
      } else if (!(base >= s.n_sink && base + kSpanRows <= all_see)) {
        products(kWhole, kRows, lds.chunk[at & 1], at, at & 1, moved_at);
      } else if (full) {
        products(kWhole, kFull, lds.chunk[at & 1], at, at & 1, moved_at);
      } else {
        products(kWhole, kPart, lds.chunk[at & 1], at, at & 1, moved_at);
      }
      moved_at = moved_at < 2 ? moved_at + 1 : 0;
    }
    __syncthreads();
    if (!loads) combine(work.chunks - 1, (work.chunks - 1) & 1, moved_at > 0 ? moved_at - 1 : 2);
  }
  if (first) {
    const int reached = (n + work.wg_rows - 1) / (work.wg_rows > 0 ? work.wg_rows : 1) * work.wg_rows;
    for (int h = 0; h < G; ++h) {
      float* vh = tab_ver + (head0 + h) * s.Lcap;
      float* sh = tab_sla + (head0 + h) * 2 * s.Lcap;
      for (int i = reached + blockIdx.x * kBatchThreads + tid; i < s.Lcap; i += gridDim.x * kBatchThreads) {
        vh[i] = 0.f;
        sh[s.Lcap + i] = 0.f;
        sh[i] = 0.f;
      }
    }
  }
  if (moments && my_head >= 0 && my_head < G) {
    stats_v.reduce_wave();
    stats_s.reduce_wave();
    if (lane == 0) {
      double x[12];
      stats_v.store(x);
      stats_s.store(x + 6);
      double* to = moments + ((head0 + my_head) * gridDim.x + blockIdx.x) * 12;
#pragma unroll
      for (int p = 0; p < 12; ++p) to[p < 4 ? p : (p < 6 ? p + 4 : (p < 10 ? p - 2 : p))] = x[p];
    }
  }
}

// One query (s = 1): its dot products are few enough to store (4 bytes per row and head beside 2 D / G of K), so the
// second pass over K is replaced by this one over them.  Vertical and slash table are equal then.  Writes the tables
// whole, and the moments of its rows as k_table_moments does.  Bound by the stores (12 bytes per row and head) and, nearly as much, by
// its instructions: 256 heads x 32K rows 28.2 us = 4.8 TB/s, 32.7 with a branch around every load and store also where a chunk lies in
// the tables whole.  grid (chunks, B*Hq), 256 threads.
constexpr int kMomentRows = 2048;
__global__ __launch_bounds__(256) void k_hist_apply_one(Shape s, float* __restrict__ tab_ver, float* __restrict__ tab_sla,
                                                        const float* __restrict__ dots, int64_t dots_stride,
                                                        const int32_t* __restrict__ seq_lens,
                                                        const float* __restrict__ part_m,
                                                        const double* __restrict__ part_l, int blocks, double gamma,
                                                        double* __restrict__ part) {
  request_arguments<decltype(&k_hist_apply_one)>();
  const int bh = blockIdx.y, b = bh / s.Hq, h = bh % s.Hq, g = h / s.G, tid = threadIdx.x;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  constexpr int U = kMomentRows / 256;
  const int row0 = blockIdx.x * kMomentRows;
  const bool whole = row0 >= s.n_sink && row0 + kMomentRows <= n;     // (then n <= Lcap covers the stores, too)
  float x[U];
  bool in[U];
  const float* from = dots + (int64_t)bh * dots_stride + row0;
  float* ver = tab_ver + (int64_t)bh * s.Lcap + row0;
  float* sla = tab_sla + (int64_t)bh * 2 * s.Lcap + row0;
  float* fresh = sla + s.Lcap;
  auto rest = [&](auto all) {
    constexpr bool kAll = decltype(all)::value;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t e = u * 256 + tid;
      const int i = row0 + (int)e;
      in[u] = kAll || (i >= s.n_sink && i < n);
      x[u] = in[u] ? from[e] : kNoScore;
    }
    float m;
    double norm;
    merge_hist<64>(part_m, part_l, ((int64_t)b * s.Hkv + g) * blocks * (kHistBatch * s.G) + h % s.G, kHistBatch * s.G,
                   blocks, tid & 63, gamma, 1, m, norm, [](float x) { return exp_below<true>(x); });
    const float hi = (float)norm, lo = (float)(norm - (double)hi);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t e = u * 256 + tid;
      x[u] = in[u] ? weigh(exp_below<true>(x[u] - m), hi, lo) : 0.f;
      if (kAll || row0 + (int)e < s.Lcap) {
        ver[e] = x[u];
        fresh[e] = x[u];
        sla[e] = 0.f;
      }
    }
  };
  if (whole) rest(std::true_type{});
  else rest(std::false_type{});
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
// K and V: 28 + 5 us at 8 groups x 32K bf16 rows (134 MB), 600 us before.  grid (splits, B*Hkv), 256 threads; 16 lanes per row, 8
// channels each, two 16-row tiles per wave in flight.
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

// The partials of a group: the sums of K and V in four blocks of 64 channels, W waves to a block, a thread every W-th partial of a
// channel with all of them on their way at once, and the scores of the heads, a wave each.  grid (B*Hkv, 5): a workgroup to
// each block and one to the scores (one workgroup for everything took 3.9 us longer for 128 partials of 8 groups: priors of 1 x 32K
// 34.7 -> 30.8 us), or kTogether: grid (B*Hkv), everything by one.
template <int W, bool kTogether>
__global__ __launch_bounds__(64 * W * (kTogether ? 4 : 1)) void k_prior_final(
    Shape s, const float* __restrict__ q, const int32_t* __restrict__ seq_lens, const double* __restrict__ part, int splits,
    float* __restrict__ kbar, float* __restrict__ vbar, float* __restrict__ sigma2_hat) {
  __shared__ double red[kTogether ? 4 : 1][W][64];
  const int bg = blockIdx.x, b = bg / s.Hkv, g = bg % s.Hkv, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const int cnt = n - s.n_sink;
  const int stride = prior_partial(s.G);
  const double* p = part + (int64_t)bg * splits * stride;
  const int mine = kTogether ? wave / W : 0, first = kTogether ? wave % W : wave;
  if (kTogether || blockIdx.y < 4) {
    const int c = 64 * (kTogether ? mine : blockIdx.y) + lane;
    double t = 0.0;
#pragma unroll 8
    for (int k = first; k < splits; k += W) t += p[(int64_t)k * stride + c];
    red[mine][first][lane] = t;
    __syncthreads();
    if (first == 0) {
      t = red[mine][0][lane];
#pragma unroll
      for (int w = 1; w < W; ++w) t += red[mine][w][lane];
      (c < kD ? kbar : vbar)[(int64_t)bg * kD + (c & (kD - 1))] = cnt > 0 ? (float)(t / (double)cnt) : 0.f;
    }
    if (!kTogether) return;
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
// Workgroups that share a KV group in k_hist_stats: 512 over all groups (lengths differ), but no more than one 128-row tile per
// wave needs.
static int hist_blocks(const Shape& s) {
  const int groups = s.B * s.Hkv;
  const int most = (s.Lcap + kHistRows * kHistWaves - 1) / (kHistRows * kHistWaves);
  int n = 512 / groups;
  n = n < 1 ? 1 : n;
  return n < most ? n : most;
}

static int moment_chunks(const Shape& s) { return (s.Lcap + kMomentRows - 1) / kMomentRows; }

// The same in the kernels of many queries, in chunks of `rows`: as many workgroups as make the least of the chunks one after the
// other, a workgroup beginning with about `wait` chunks' worth of waiting for its first rows and queries.  A CU takes one workgroup at a
// time (pair 0), or two, which together take pair / 20 times as long.  merge: twentieths of a chunk that 32 workgroups of a group cost
// whoever reads their results (merge_hist: eight loads of each of four lanes at a time).
static int batch_blocks(const Shape& s, int rows, int wait, int pair, int merge) {
  const int64_t groups = (int64_t)s.B * s.Hkv, tiles = (s.Lcap + rows - 1) / rows, slots = pair ? 512 : 256;
  int64_t best = 1, least = INT64_MAX;
  for (int64_t n = 1; n <= tiles && n <= slots; ++n) {
    const int64_t all = groups * n, rest = all % slots;
    const int64_t rounds = all / slots * (pair ? pair : 20) + (rest > 256 ? pair : (rest > 0 ? 20 : 0));  // in twentieths
    const int64_t cost = rounds * ((tiles + n - 1) / n + wait) + (n + 31) / 32 * merge;
    if (cost < least) {
      least = cost;
      best = n;
    }
  }
  return (int)best;
}
// Every workgroup of the second kernel reads all partials of its group before its first product: 32 queries of one group (four heads) x
// 128K rows with 512 of them 85.3 us, 256 61.6, 192 59.3, 128 58.4 (two queries 39.4, 31.1, 32.1, 33.1), of 8 groups x 32K with 64 71.6,
// 32 65.6, of 8 x 128K with 64 208, 32 219.
HistPlan plan_table_history(const Shape& s) {
  HistPlan plan;
  plan.parts[kPartsShort] = batch_blocks(s, 64, 4, 35, 62);
  plan.parts[kPartsOneUnit] = batch_blocks(s, 128, 4, 35, 62);
  plan.parts[kPartsFp8] = batch_blocks(s, 128, 2, 35, 31);             // (the same waits in chunks of twice the rows)
  plan.blocks = batch_blocks(s, kApplyRows, 2, 0, 0);
  return plan;
}

int64_t table_init_scratch_bytes(const Shape& s, const HistPlan& plan) {
  int most = hist_blocks(s);
  for (int p : plan.parts) most = p > most ? p : most;
  const int parts = moment_chunks(s) > plan.blocks ? moment_chunks(s) : plan.blocks;
  return (int64_t)s.B * s.Hkv * most * kHistBatch * s.G * (8 + 4) + (int64_t)s.B * s.Hq * parts * 12 * 8;
}

// Up to how many bytes of keys the first pass over K reads with ordinary loads.  Keys that will not be found in the memory-side cache
// again are read past it (one query, 64 groups x 32K rows, 537 MB: 119 -> 96 us).  With one query the next reader is the next call, and
// the tables, written whole in between, take their part of the cache: tables of 4 x capacity, K + tables 224 MB 54.2 us kept, 58.4 past
// the caches, 280 MB 74.0 and 72.8, 336 MB 91.2 and 79.1.  With more queries k_batch_apply reads the keys again at once, while it writes
// the tables.  Kept and past the caches, 4 queries (16 and 32 much the same), MiB of keys + tables: bf16 256 + 48 101.6 and 125.6, 320 +
// 60 143.5 and 139.3, 512 + 96 244.2 and 218.8; fp16, two heads per group, 320 + 30 132.9 and 135.2, 448 + 42 189.6 and 187.0; bf16, one
// head, 384 + 18 152.0 and 155.0, 512 + 24 223.1 and 214.8; FP8 keys 224 + 84 146.9 and 146.1, 256 + 96 145.6 and 146.0, 320 + 120 195.8
// and 183.7.  That second pass keeps ordinary loads: past the caches 257 us instead of 251 at 268 + 100 MB, 481 instead of 476 at 537 +
// 200 MB, both passes.
static float stats_kept_bytes(const Shape& s, int n_queries) {
  const float tables = 12.f * s.B * s.Hq * s.Lcap;
  return n_queries == 1 ? (float)kKeptBytes - tables : 440.f * (1 << 20) - 2.4f * tables;
}

// The units of a batch of nq queries as the kernels are built for them.  (What the quads of a chunk move up, 4 rows for each before
// the last and 15 for the rows, has to end in the next one.)  One unit of grouped heads: over FP8 keys, where a wave's products then
// take half as long beside the conversion of the rows, 2 queries with one unit instead of two (one of them without a query): 64 groups
// (two heads each) x 16000 rows 79.6 -> 67.5 us, 8 x 32K 32.8 -> 28.7, four heads each 74.6 -> 68.3 and 32.6 -> 30.2.  (128 x
// 32K, past the caches, 265 -> 280.)  Over 16-bit keys the longer chunks that one unit needs in the first kernel cost more: 8 x 32K bf16
// 36.4 -> 39.0, 64 x 16000 96.7 -> 102.7.
static int batch_units(int G, int nq, int kind) {
  const int units = ((nq + 3) / 4 * G + 3) / 4;
  return units == 1 && G > 1 && kind != kKindFp8 ? 2 : (units == 3 ? 4 : (units > 4 ? 8 : units));
}

// X(heads per group, units, key format)
#define LFPS_BATCH_FOR_EACH_U(X, KIND) X(4, 2, KIND) X(4, 4, KIND) X(4, 8, KIND) X(2, 2, KIND) X(2, 4, KIND) X(1, 1, KIND) X(1, 2, KIND)
#define LFPS_BATCH_FOR_EACH(X)                                                                                            \
  LFPS_BATCH_FOR_EACH_U(X, kKindBf16) LFPS_BATCH_FOR_EACH_U(X, kKindFp8) LFPS_BATCH_FOR_EACH_U(X, kKindF16)               \
  X(4, 1, kKindFp8) X(2, 1, kKindFp8)

// Called once per context in table mode: the second kernel needs more dynamic LDS than the default limit.
hipError_t configure_table_history(const Shape& s, int k_kind) {
  hipError_t e = hipSuccess;
  auto raise = [&](const void* kernel, int bytes) {
    if (e == hipSuccess) e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  };
#define LFPS_RAISE_BATCH(GG, UU, KIND)                                                       \
  if (s.G == GG && k_kind == KIND) {                                                         \
    raise((const void*)k_batch_apply<GG, false, KIND, UU>, (int)sizeof(ApplyLds<UU>));       \
    raise((const void*)k_batch_apply<GG, true, KIND, UU>, (int)sizeof(ApplyLds<UU>));        \
  }
  LFPS_BATCH_FOR_EACH(LFPS_RAISE_BATCH)
#undef LFPS_RAISE_BATCH
  return e;
}

// What the launches below share.  The scratch: moments, then the partials of the statistics.
struct HistScratch {
  double* moments;
  double* part_l;
  float* part_m;
  HistScratch(const Shape& s, void* scratch, int blocks, int parts) {
    moments = static_cast<double*>(scratch);
    part_l = moments + (int64_t)s.B * s.Hq * parts * 12;
    part_m = reinterpret_cast<float*>(part_l + (int64_t)s.B * s.Hkv * blocks * kHistBatch * s.G);
  }
};

template <int G, bool kPaged, int kKind, int U>
static hipError_t launch_batch_t(const Shape& s, const HistPlan& plan, float* tab_ver, float* tab_sla, const float* q0, int64_t q_stride, int j0,
                                 int nq, int n_queries, double gamma, const KvView& kv, void* scratch, int32_t* flags,
                                 hipStream_t st) {
  const int parts = plan.parts[stats_form(U, kKind)], blocks = plan.blocks;
  const HistScratch to(s, scratch, parts, blocks);
  const dim3 block(kBatchThreads);
  const float kept = stats_kept_bytes(s, n_queries);
  hipLaunchKernelGGL((k_batch_stats<G, kPaged, kKind, U>), dim3(parts, s.B * s.Hkv), block, 0, st, s, q0, q_stride, j0, nq, kv.k, kv.stride_b,
                     kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, to.part_m, to.part_l, flags, kept);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_batch_apply<G, kPaged, kKind, U>), dim3(blocks, s.B * s.Hkv), block, sizeof(ApplyLds<U>), st, s, tab_ver, tab_sla, q0, q_stride,
                     j0, nq, kv.k, kv.stride_b, kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, to.part_m, to.part_l, parts, gamma,
                     n_queries, n_queries <= kHistBatch ? to.moments : nullptr);
  return hipGetLastError();
}

static hipError_t launch_batch(const Shape& s, const HistPlan& plan, float* tab_ver, float* tab_sla, const float* q0, int64_t q_stride, int j0,
                               int nq, int n_queries, double gamma, const KvView& kv, void* scratch, int32_t* flags,
                               hipStream_t st) {
  const int kind = kv.k_fp8 ? kKindFp8 : (kv.f16 ? kKindF16 : kKindBf16), units = batch_units(s.G, nq, kind);
#define LFPS_HIST_ARGS s, plan, tab_ver, tab_sla, q0, q_stride, j0, nq, n_queries, gamma, kv, scratch, flags, st
#define LFPS_LAUNCH_BATCH(GG, UU, KIND)                                                      \
  if (s.G == GG && units == UU && kind == KIND)                                              \
    return kv.page.table ? launch_batch_t<GG, true, KIND, UU>(LFPS_HIST_ARGS)                \
                         : launch_batch_t<GG, false, KIND, UU>(LFPS_HIST_ARGS);
  LFPS_BATCH_FOR_EACH(LFPS_LAUNCH_BATCH)
#undef LFPS_LAUNCH_BATCH
#undef LFPS_HIST_ARGS
  return hipErrorInvalidValue;
}

template <int G, bool kPaged, int kKind>
static hipError_t launch_one_t(const Shape& s, float* tab_ver, float* tab_sla, const float* q, double gamma, const KvView& kv,
                               float* dots, int64_t dots_stride, void* scratch, int32_t* flags, hipStream_t st) {
  const int blocks = hist_blocks(s), chunks = moment_chunks(s);
  const HistScratch to(s, scratch, blocks, chunks);
  const float kept = stats_kept_bytes(s, 1);
#define LFPS_STATS(ONCE)                                                                                                \
  hipLaunchKernelGGL((k_hist_stats<G, kPaged, kKind, ONCE>), dim3(blocks, s.B * s.Hkv), dim3(kHistWaves * 64), 0, st, s, q, \
                     kv.k, kv.stride_b, kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, to.part_m, to.part_l, dots,      \
                     dots_stride, flags, kept)
  if ((float)s.B * s.Hkv * s.Lcap * (kD * KSub<kKind>::kElemBytes) > kept) LFPS_STATS(true);
  else LFPS_STATS(false);
#undef LFPS_STATS
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_hist_apply_one, dim3(chunks, s.B * s.Hq), dim3(256), 0, st, s, tab_ver, tab_sla, dots, dots_stride,
                     kv.seq_lens, to.part_m, to.part_l, blocks, gamma, to.moments);
  return hipGetLastError();
}

static hipError_t launch_one(const Shape& s, float* tab_ver, float* tab_sla, const float* q, double gamma, const KvView& kv,
                             float* dots, int64_t dots_stride, void* scratch, int32_t* flags, hipStream_t st) {
#define LFPS_HIST_ARGS s, tab_ver, tab_sla, q, gamma, kv, dots, dots_stride, scratch, flags, st
#define LFPS_HIST(GG, KIND)                                                        \
  return kv.page.table ? launch_one_t<GG, true, KIND>(LFPS_HIST_ARGS)              \
                       : launch_one_t<GG, false, KIND>(LFPS_HIST_ARGS)
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

hipError_t launch_table_history(const Shape& s, const HistPlan& plan, float* tab_ver, float* tab_sla, const float* q_hist, int n_queries,
                                double gamma, const KvView& kv, float* dots, int64_t dots_stride, void* scratch,
                                int32_t* flags, int* moment_parts, hipStream_t st) {
  if (n_queries == 1) {
    *moment_parts = moment_chunks(s);
    return launch_one(s, tab_ver, tab_sla, q_hist, gamma, kv, dots, dots_stride, scratch, flags, st);
  }
  const int64_t q_stride = (int64_t)s.B * s.Hq * kD;
  for (int j0 = 1; j0 <= n_queries; j0 += kHistBatch) {
    const int nq = n_queries - j0 + 1 < kHistBatch ? n_queries - j0 + 1 : kHistBatch;
    const hipError_t e = launch_batch(s, plan, tab_ver, tab_sla, q_hist + (int64_t)(j0 - 1) * q_stride, q_stride, j0, nq, n_queries,
                                      gamma, kv, scratch, flags, st);
    if (e != hipSuccess) return e;
  }
  *moment_parts = n_queries <= kHistBatch ? plan.blocks : 0;
  return hipSuccess;
}

hipError_t launch_table_state(const Shape& s, const float* tab_ver, const float* tab_sla, double* state,
                              const int32_t* seq_lens, void* scratch, int moment_parts, hipStream_t st) {
  double* part = static_cast<double*>(scratch);
  if (!moment_parts) {
    moment_parts = moment_chunks(s);
    hipLaunchKernelGGL(k_table_moments, dim3(moment_parts, s.B * s.Hq), dim3(256), 0, st, s, tab_ver, tab_sla, seq_lens, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_table_state, dim3(s.B * s.Hq), dim3(192), 0, st, s, part, moment_parts, state, seq_lens);
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
#define LFPS_LAUNCH_FINAL(W, TOGETHER)                                                                                  \
  hipLaunchKernelGGL((k_prior_final<W, TOGETHER>), dim3(s.B * s.Hkv, TOGETHER ? 1 : 5), dim3(64 * W * (TOGETHER ? 4 : 1)), 0, \
                     st, s, q, kv.seq_lens, part, splits, kbar, vbar, sigma2_hat)
  // From 256 groups on (four partials each) as many workgroups as groups: 1024 groups x 1000 rows 109.7 us, with five of sixteen waves
  // each 116.1, five of four 112.3; 512 x 2000 103.4, 109.1.  Up to sixteen partials four waves: 64 x 4000 30.9 -> 29.9.
  if (s.B * s.Hkv >= 256) LFPS_LAUNCH_FINAL(4, true);
  else if (splits > 16) LFPS_LAUNCH_FINAL(16, false);
  else LFPS_LAUNCH_FINAL(4, false);
#undef LFPS_LAUNCH_FINAL
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
