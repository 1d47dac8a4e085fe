// The MFMA scoring arithmetic shared by the kernels that score K rows against the G query heads of a KV group
// (Alg. 1 line 8; Sec. 1 Step 1): the three-term split of the fp32 query, the register tile of K rows, and the loop
// that scores a strided set of a group's candidate slots.  One definition, so that a row's score is the same bits
// whichever kernel computes it.
#pragma once
#include "lfps_internal.h"

#include <float.h>

#include <type_traits>

namespace lfps {

constexpr int kScoreThreads = 256;           // 4 waves
constexpr int kRowsPerWaveIter = 64;         // rows a wave scores per loop iteration

// Storage format of the K rows a scoring kernel reads.
enum { kKindBf16 = 0, kKindFp8 = 1, kKindF16 = 2 };

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Term t (0, 1, 2; 3: zeros) of the three-way split of eight fp32 query elements into the operand's 16-bit format, and the
// sum of the three MFMA results that undoes the split.  Every wave of a scoring kernel splits 32 elements per lane before
// its first product, so this is kept short: two elements per hardware conversion (round to nearest even), and the term is
// chosen by factors of 0 and 1, without branches: 7 instructions an element (rounding in integer arithmetic took about 30;
// with selects, which the compiler made branches, four steps of 1 x 32K took 109 us instead of 106, of 3 x 20K fp16 92 instead
// of 87).  An infinite or overflowing element makes NaNs here or in the sum, as a difference of infinities does.
template <typename Op>
struct Split3;
template <>
struct Split3<bf16x8> {
  static constexpr bool kHalf = false;
  __device__ static __forceinline__ bf16x8 terms(const float (&f)[8], int t) {
    bf16x8 out;
    const float one = t >= 1 ? -1.f : 0.f, two = t >= 2 ? -1.f : 0.f;      // (no branches: the lanes of a wave make different terms)
#pragma unroll
    for (int c = 0; c < 8; c += 2) {
      f32x2 x = {f[c], f[c + 1]};
      f32x2 y = __builtin_convertvector(__builtin_convertvector(x, bf16x2), f32x2);
      x = {fmaf(one, y[0], x[0]), fmaf(one, y[1], x[1])};
      y = __builtin_convertvector(__builtin_convertvector(x, bf16x2), f32x2);
      x = {fmaf(two, y[0], x[0]), fmaf(two, y[1], x[1])};
      const bf16x2 b = __builtin_convertvector(x, bf16x2);
      out[c] = t < 3 ? b[0] : (__bf16)0.f;
      out[c + 1] = t < 3 ? b[1] : (__bf16)0.f;
    }
    return out;
  }
  __device__ static __forceinline__ float sum(const f32x4& acc) { return (acc[0] + acc[1]) + acc[2]; }
};
template <>
struct Split3<f16x8> {
  static constexpr bool kHalf = true;
  // q = t0 + t1 / 2^11 + t2 / 2^22 (11 significant bits per term; the scaling keeps t1, t2 normal)
  __device__ static __forceinline__ f16x8 terms(const float (&f)[8], int t) {
    f16x8 out;
    const float one = t >= 1 ? -1.f : 0.f, two = t >= 2 ? -1.f / 2048.0f : 0.f;
    const float up = t == 0 ? 1.f : (t == 1 ? 2048.0f : 4194304.0f), up1 = t >= 2 ? 2048.0f : 0.f;   // (0: a large x must not overflow)
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      float x = fmaf(one, (float)(_Float16)f[c], f[c]);
      x = fmaf(two, (float)(_Float16)(x * up1), x);
      const _Float16 h = (_Float16)(x * up);
      out[c] = t < 3 ? h : (_Float16)0.0f;
    }
    return out;
  }
  __device__ static __forceinline__ float sum(const f32x4& acc) {
    return (acc[0] + acc[1] * (1.0f / 2048.0f)) + acc[2] * (1.0f / 4194304.0f);
  }
};

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma16(f16x8 a, f16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// The MFMA A operand of lane (j, kb): row m = j of the 16x32 A tile of step kk holds term (m & 3)
// of head (m >> 2), channels of the 16-byte chunk kk + 4*kb of the row (the chunk that lane group kb
// loads from K at step kk).  Heads >= G contribute zeros.  The query is fetched with eight 16-byte
// loads issued together; a lane-dependent branch here would serialise 32 single loads.
// Returns true if this lane met a query element beyond the fp16 range (fp16 operands only): the element is
// clamped to +-65504 so that the scores stay finite, and the caller raises LFPS_FLAG_Q_RANGE.
// (In two parts for callers that have rows to request between the query's arrival and its use.)
struct QueryRows {
  float4 x[4][2];
  __device__ __forceinline__ void load(const float* __restrict__ q, int64_t head0, int G, int j, int kb) {
    const int h = j >> 2;
    const float4* qh = reinterpret_cast<const float4*>(q + (head0 + (h < G ? h : 0)) * kD);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      x[kk][0] = qh[2 * (kk + 4 * kb)];
      x[kk][1] = qh[2 * (kk + 4 * kb) + 1];
    }
  }
  template <typename Op>
  __device__ __forceinline__ bool operand(Op (&A)[4], int G, int j) const {
    const int h = j >> 2, t = j & 3;
    const bool live = h < G && t < 3;
    bool clipped = false;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      float f[8] = {x[kk][0].x, x[kk][0].y, x[kk][0].z, x[kk][0].w, x[kk][1].x, x[kk][1].y, x[kk][1].z, x[kk][1].w};
      if constexpr (Split3<Op>::kHalf) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          if (fabsf(f[c]) > 65504.0f) {               // also +-inf; a NaN goes through as in the other formats
            clipped |= live;
            f[c] = copysignf(65504.0f, f[c]);
          }
        }
      }
      A[kk] = Split3<Op>::terms(f, live ? t : 3);
    }
    return clipped;
  }
};
template <typename Op>
__device__ __forceinline__ bool load_query_operand(Op (&A)[4], const float* __restrict__ q, int64_t head0, int G, int j,
                                                   int kb) {
  QueryRows rows;
  rows.load(q, head0, G, j, kb);
  return rows.operand(A, G, j);
}

// One lane of the wave reports a clamped query element (fp16 caches only; compiled out otherwise).
__device__ __forceinline__ void report_q_range(bool clipped, int32_t* __restrict__ flags) {
  if (__ballot(clipped) != 0 && (threadIdx.x & 63) == 0) atomicOr(flags, LFPS_FLAG_Q_RANGE);
}

// The registers a lane (j, kb) holds of 16 K rows: its 32 channels [32 kb, 32 kb + 32) of row j, in the storage format
// of K.  operand(kk) is the MFMA B operand of step kk, the channels 32 kb + 8 kk .. + 7 as bf16: the value as stored for
// a bf16 cache, converted (exactly: every E4M3 value is a bf16 value) when it is multiplied for an FP8 cache, so that
// a tile in flight costs half the registers and half the loads.
template <int kKind>
struct KSub;
template <>
struct KSub<kKindBf16> {
  using Operand = bf16x8;
  static constexpr int kElemBytes = 2;
  bf16x8 v[4];
  __device__ __forceinline__ void load_row(const char* row, int kb) {
    const bf16x8* p = reinterpret_cast<const bf16x8*>(row) + 4 * kb;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) v[kk] = p[kk];
  }
  __device__ __forceinline__ bf16x8 operand(int kk) const { return v[kk]; }
};
template <>
struct KSub<kKindF16> {
  using Operand = f16x8;
  static constexpr int kElemBytes = 2;
  f16x8 v[4];
  __device__ __forceinline__ void load_row(const char* row, int kb) {
    const f16x8* p = reinterpret_cast<const f16x8*>(row) + 4 * kb;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) v[kk] = p[kk];
  }
  __device__ __forceinline__ f16x8 operand(int kk) const { return v[kk]; }
};
template <>
struct KSub<kKindFp8> {
  using Operand = bf16x8;
  static constexpr int kElemBytes = 1;
  u32x4 v[2];
  __device__ __forceinline__ void load_row(const char* row, int kb) {
    const u32x4* p = reinterpret_cast<const u32x4*>(row) + 2 * kb;
    v[0] = p[0];
    v[1] = p[1];
  }
  __device__ __forceinline__ bf16x8 operand(int kk) const {
    const u32x4 w = v[kk >> 1];
    return (kk & 1) ? fp8x8_to_bf16x8(w[2], w[3]) : fp8x8_to_bf16x8(w[0], w[1]);
  }
};

// The value of x in lane `base + more` of the wave (more: known when compiled; it becomes the instruction's offset).
__device__ __forceinline__ int lane_value(int x, int base, int more) {
  return __builtin_amdgcn_ds_bpermute(4 * base + 4 * more, x);
}

// A 64-row K tile: sub-tile t holds the rows 16 t + j, every lane loads its own channels of its row (four loads touch every
// cache line of a row).
template <int kKind>
struct KTile {
  using Operand = typename KSub<kKind>::Operand;
  static constexpr int kElemBytes = KSub<kKind>::kElemBytes;
  KSub<kKind> s_[4];
  __device__ __forceinline__ void load_row(int t, const char* row, int kb) { s_[t].load_row(row, kb); }
  __device__ __forceinline__ Operand operand(int t, int kk) const { return s_[t].operand(kk); }
  // the rows whose addresses relative to Kbg are offset(lane's row id of that tile row)
  template <typename Offset>
  __device__ __forceinline__ void fetch(const char* Kbg, int phys, int lane, Offset offset) {
#pragma unroll
    for (int t = 0; t < 4; ++t) load_row(t, Kbg + offset(lane_value(phys, lane & 15, 16 * t)), lane >> 4);
  }
  __device__ __forceinline__ KSub<kKind> sub(int t, u32x4*, int) const { return s_[t]; }
};

// The same tile fetched past the caches: every load instruction of the wave covers whole rows (16 lanes a row, 8 of FP8), so
// that a cache line is touched by one instruction only and need not be kept (non-temporal).  sub(t) turns the sixteen rows of
// sub-tile t into operands through a wave-private piece of LDS (rows 16 bytes further apart than they are long, so that
// neither the writes nor the reads of neighbouring lanes meet in a bank): the operands, and so the scores' bits, are KTile's.
// once false: the same instructions with ordinary loads.
template <int kKind>
struct StreamTile {
  using Operand = typename KSub<kKind>::Operand;
  static constexpr int kElemBytes = KSub<kKind>::kElemBytes;
  static constexpr int kChunks = kD * kElemBytes / 16;                 // of a row
  static constexpr int kLoadRows = 64 / kChunks;                       // rows of a load instruction
  static constexpr int kLoads = kRowsPerWaveIter / kLoadRows;
  static constexpr int kLdsChunks = 16 * (kChunks + 1);
  u32x4 raw[kLoads];
  template <typename Offset>
  __device__ __forceinline__ void fetch(const char* Kbg, int phys, int lane, Offset offset, bool once = true) {
    const u32x4* mine = reinterpret_cast<const u32x4*>(Kbg) + lane % kChunks;
    auto at = [&](int i) {
      const int row = lane_value(phys, lane / kChunks, i * kLoadRows);
      return reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(mine) + offset(row));
    };
    if (once) {
      asm volatile("; past the caches");                               // (or the compiler makes ordinary loads of both branches)
#pragma unroll
      for (int i = 0; i < kLoads; ++i) raw[i] = __builtin_nontemporal_load(at(i));
      asm volatile("; past the caches");
    } else {
#pragma unroll
      for (int i = 0; i < kLoads; ++i) raw[i] = *at(i);
    }
  }
  __device__ __forceinline__ KSub<kKind> sub(int t, u32x4* lds, int lane) const {
    constexpr int kPer = kLoads / 4, kPitch = kChunks + 1;
    u32x4* to = lds + lane / kChunks * kPitch + lane % kChunks;
    const u32x4* from = lds + (lane & 15) * kPitch + kChunks / 4 * (lane >> 4);
    wave_lds_order();                                                  // the reads of the sub-tile before
#pragma unroll
    for (int i = 0; i < kPer; ++i) to[i * kLoadRows * kPitch] = raw[kPer * t + i];
    wave_lds_order();
    KSub<kKind> out;
#pragma unroll
    for (int c = 0; c < kChunks / 4; ++c) out.v[c] = __builtin_bit_cast(std::remove_reference_t<decltype(out.v[0])>, from[c]);
    return out;
  }
};

// Scores of the slots first .. first+63, first+step .. first+step+63, ... (below count) of one KV group, by one wave:
// lane (j, kb) = (lane & 15, lane >> 4) loads the chunks of K that lane group kb owns and ends up holding head kb's
// score of slot base + 16 t + j.  row_at(slot): its row position.  A slot whose position lies outside [0, n) reads row 0 and scores -inf: it ranks below every row.
// The row ids of the next visit are fetched, and the scores of the previous visit stored, right after this visit's
// loads are issued.  sc: the score row of head kb (ignored by lanes with store == false).
// tops (or NULL): receives the largest score of every 16 slots, as the select orders them (a NaN above all); first and step are
// multiples of 64 then.
// turn (or NULL, see kStream): a wave-private piece of LDS, through which the rows come as whole ones (StreamTile, ordinary loads; the
// same bits).  query (or NULL): the rows A is made from, here, behind the requests for the first tile.  (k_sample_score.)
template <bool kPaged, int kKind, bool kTops = false, bool kStream = false, typename RowAt>
__device__ __forceinline__ void score_slots_mfma(typename KTile<kKind>::Operand (&A)[4], const char* Kbg,
                                                 const KvPage& pg, int b, int64_t stride_b, int64_t stride_n,
                                                 RowAt row_at, int n, int count, int first, int step,
                                                 float* __restrict__ sc, bool store, float scale,
                                                 float* __restrict__ tops = nullptr, u32x4* turn = nullptr,
                                                 const QueryRows* query = nullptr, int G = 0, int32_t* flags = nullptr) {
  using Rows = RowMap<kPaged>;
  using Op = typename KTile<kKind>::Operand;
  constexpr int ES = KTile<kKind>::kElemBytes;
  const int lane = threadIdx.x & 63, j = lane & 15;
  auto valid = [&](int row) { return row >= 0 && row < n; };
  auto physical = [&](int row) { return Rows::phys(pg, b, valid(row) ? row : 0); };

  float pv[4] = {0.f, 0.f, 0.f, 0.f};   // scores of the previous visit, not yet stored
  int pbase = -1;
  int my_row = -1;
  if (first + lane < count) my_row = row_at(first + lane);
  int my_ok = valid(my_row);
  my_row = physical(my_row);
  for (int base = first; base < count; base += step) {
    std::conditional_t<kStream, StreamTile<kKind>, KTile<kKind>> Bt;
    bool ok_t[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) ok_t[t] = __shfl(my_ok, 16 * t + j) != 0;
    auto offset = [&](int row) { return Rows::offset(pg, row, stride_b, stride_n) * ES; };
    if constexpr (kStream) Bt.fetch(Kbg, my_row, lane, offset, false);
    else Bt.fetch(Kbg, my_row, lane, offset);
    if (query && base == first) {
      __builtin_amdgcn_sched_barrier(0);
      report_q_range(query->operand(A, G, j), flags);
    }
    const int nb = base + step;
    int next_row = -1;
    if (nb + lane < count) next_row = row_at(nb + lane);
    const int next_ok = valid(next_row);
    next_row = physical(next_row);
    if (pbase >= 0) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int slot = pbase + 16 * t + j;
        if (store && slot < count) sc[slot] = pv[t];
      }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const KSub<kKind> sub = Bt.sub(t, turn, lane);
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        acc = mfma16(A[kk], sub.operand(kk), acc);
      // lane (j, kb): D rows 4*kb .. 4*kb+3 = the three terms (and a zero row) of head kb, column j
      pv[t] = ok_t[t] ? Split3<Op>::sum(acc) * scale : -INFINITY;
    }
    if constexpr (kTops) {
      if (tops) {
        float mine = 0.f;                                  // lane j: of the slots 16 j .. 16 j + 15, j < 4
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float x = base + 16 * t + j < count ? fmaxf(fminf(pv[t], FLT_MAX), -FLT_MAX) + 0.0f : -FLT_MAX;
          const float top = row16_max(x);
          mine = j == t ? top : mine;
        }
        if (store && j < 4 && base + 16 * j < count) tops[(base >> 4) + j] = mine;
      }
    }
    pbase = base;
    my_row = next_row;
    my_ok = next_ok;
  }
  if (pbase >= 0) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int slot = pbase + 16 * t + j;
      if (store && slot < count) sc[slot] = pv[t];
    }
  }
}

}  // namespace lfps
