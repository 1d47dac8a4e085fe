// Score tables of LFPS (Sec. 4.2: Eq. 4 initialisation, Eq. 7-8 thresholds, Eq. 10 update; App. B.2).
//
// Per query head two tables over positions, vertical and slash.  Eq. 10 decays every entry by gamma each
// step, moves slash history from i-1 to i, and adds (w_i - 1/(2|C_2|)) on the selected positions only.
// Stored so that a step touches the selected entries and nothing else:
//   * scale: a table entry is  Phi(i) = g * A(i)  with one factor g per head.  The decay is g <- gamma g;
//     a selected entry becomes A(i) += delta_i / (gamma g).  (When g gets small a dense pass
//     folds it back into A, at the end of the update that made it small; each head decides for itself.)
//   * slash frame: A_sla is stored at index  i - cnt + Lcap  (cnt = updates applied so far), so the move
//     of history from i-1 to i is the increment of cnt.  The entry of a new position is the slot its
//     predecessor had; position 0 moves onto a slot that was never written (zero).
//   * statistics: Eq. 8 needs the mean, sum (x-mean)^2 and sum (x-mean)^4 of each table.  The raw
//     moments M_p = sum x^p (p = 1..4, fp64) follow the update exactly: M_p <- gamma^p M_p +
//     sum over selected of ((gamma x + delta)^p - (gamma x)^p); a new position adds a zero.
//     The thresholds of a step are derived from them when its scan starts.
// Sink positions (< n_sink) are outside the tables: never flagged, counted or updated.
//
// The only dense work of a step is the scan (k_table_flags): both tables are read once and two bits
// per position and head are written (initial candidate; above the mean).
#include "lfps_internal.h"

#include <type_traits>

namespace lfps {

constexpr int kTabThreads = 256;
constexpr int kFlagIters = 8;      // 64-position tests per wave of the scan kernel
constexpr double kFoldBelow = 1e-20;   // gamma = 0.95 gets here after ~900 updates; stored values stay < 1e20 * Phi

// The update count as stored (a double) brought into [0, Lcap - 1]: every slash-frame index formed with
// it stays inside the table's 2 * Lcap slots (the host refuses updates beyond that count).
__device__ __forceinline__ int clamp_count(double c, int Lcap) {
  const int v = (int)c;
  return v < 0 ? 0 : (v > Lcap - 1 ? Lcap - 1 : v);
}

__device__ __forceinline__ double block_sum(double v, double* red, int tid) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) v += __shfl_xor(v, d);
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < (int)blockDim.x / 64; ++w) t += red[w];
  return t;
}

__device__ __forceinline__ float block_min(float v, float* red, int tid) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) v = fminf(v, __shfl_xor(v, d));
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  float t = red[0];
  for (int w = 1; w < (int)blockDim.x / 64; ++w) t = fminf(t, red[w]);
  return t;
}

// Eq. 8 from raw moments over N entries: thresholds and means in true units.
__device__ __forceinline__ void thresholds_from_moments(const double* M, double N, double a, bool flat, double* tau,
                                                        double* mean) {
  if (N <= 0.0) {
    *tau = INFINITY;
    *mean = 0.0;
    return;
  }
  const double m = M[0] / N;
  *mean = m;
  const double c2 = M[1] - N * m * m;
  const double c4 = M[3] - 4.0 * m * M[2] + 6.0 * m * m * M[1] - 3.0 * N * m * m * m * m;
  if (flat || !(c2 > 0.0) || !(c4 > 0.0)) {
    *tau = INFINITY;                        // no pattern: nothing exceeds the threshold
    return;
  }
  const double kappa = c4 / (c2 * c2);
  *tau = a * m / kappa;
}

// ----------------------------------------------------------------------------- scan (Eq. 7, Eq. 9 predicates)
// Largest float <= t (t finite or +inf; NaN gives +inf: nothing passes).  For a float x and a double
// threshold t:  x > t  <=>  x > float_below(t), so the scan can compare in fp32 without changing a decision.
__device__ __forceinline__ float float_below(double t) {
  if (!(t == t)) return INFINITY;
  float f = (float)t;                                   // round to nearest
  if ((double)f > t) f = nextafterf(f, -INFINITY);
  return f;
}

// grid (chunks, B*Hq).  Each wave tests 64 consecutive positions per iteration; the ballots are the
// flag words.  A table entry is g * A(i); the comparison  g * A > threshold  is made as  A > threshold / g
// with the quotient (fp64) rounded down to fp32 once per workgroup: by one wave, the vertical table's in its even lanes
// and the slash table's in its odd ones, behind the requests for the first rows.  Bound by the bytes of both tables, of
// which 256 heads x 32K rows (a fifth of the heads bypassed) take 54 MB: 11.8 us = 4.6 TB/s.  14.8 us with the quotients
// found by every wave, one table after the other and before the requests, and a branch around each load and comparison.
__global__ __launch_bounds__(kTabThreads) void k_table_flags(Shape s, const float* __restrict__ tab_ver,
                                                             const float* __restrict__ tab_sla,
                                                             const double* __restrict__ state,
                                                             const int32_t* __restrict__ seq_lens,
                                                             uint32_t* __restrict__ f0, uint32_t* __restrict__ fm,
                                                             int flag_words, int rows_per_block, double a,
                                                             const int32_t* __restrict__ gate) {
  request_arguments<decltype(&k_table_flags)>();
  __shared__ uint32_t w0[kFlagIters * kTabThreads / 32], wm[kFlagIters * kTabThreads / 32];
  __shared__ float limits[4];                             // threshold and mean of the vertical, then of the slash table
  const int bh = blockIdx.y, b = bh / s.Hq;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const double* st = state + (int64_t)bh * kTableStateDoubles;
  // everything that depends on the head alone in one round trip (the gate's word, too: without a gate any other is read)
  const int gate_word = *(gate ? gate + bh : seq_lens + b);
  const double moves = st[TS_CNT], g = st[TS_G], flat_n = st[TS_FLAT_N];
  int n = seq_lens[b];
  const bool slash = lane & 1;
  double M[4], flat = 0.0;
  if (wave == 0) {
#pragma unroll
    for (int p = 0; p < 4; ++p) M[p] = st[(slash ? TS_MS : TS_MV) + p];
    flat = st[slash ? TS_FLAT_S : TS_FLAT_V];
  }
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const int n_round = (n + 63) & ~63;                     // whole flag words up to the end of the sequence
  asm volatile("" ::"s"(moves), "s"(g), "s"(flat_n));     // (the compiler would ask for them behind the branch)
  if (gate && gate_word != 0) {                           // bypassed head: it proposes no candidates
    const int w_begin = (blockIdx.x * rows_per_block) >> 5;
    const int w_end = ((blockIdx.x + 1) * rows_per_block < n_round ? (blockIdx.x + 1) * rows_per_block : n_round) >> 5;
    for (int w = w_begin + tid; w < w_end; w += kTabThreads) {
      f0[(int64_t)bh * flag_words + w] = 0u;
      fm[(int64_t)bh * flag_words + w] = 0u;
    }
    return;
  }
  const int cnt = clamp_count(moves, s.Lcap);
  const float* ver = tab_ver + (int64_t)bh * s.Lcap;
  const float* sla = tab_sla + (int64_t)bh * 2 * s.Lcap + (s.Lcap - cnt);
  uint32_t* o0 = f0 + (int64_t)bh * flag_words;
  uint32_t* om = fm + (int64_t)bh * flag_words;
  float tau_v = 0.f, tau_s = 0.f, mean_v = 0.f, mean_s = 0.f;
  auto find_limits = [&]() {
    if (wave == 0) {
      const double N = (double)(n - s.n_sink > 0 ? n - s.n_sink : 0);
      double t, m;
      thresholds_from_moments(M, N, a, flat != 0.0 && (flat_n == N || M[1] == 0.0), &t, &m);
      const float tau = float_below(t / g), mean = float_below(m / g);
      if (lane < 2) {
        limits[2 * lane] = tau;
        limits[2 * lane + 1] = mean;
      }
    }
    __syncthreads();
    tau_v = limits[0];
    mean_v = limits[1];
    tau_s = limits[2];
    mean_s = limits[3];
  };
  // A workgroup covers rows_per_block consecutive positions in passes of kFlagIters * 256; in a pass wave w
  // takes every fourth 64-position word pair, and all its loads are issued before the first comparison
  // (fixed trip count, fully unrolled).  The flag words of a pass meet in LDS and leave as two coalesced stores.
  constexpr int kPassRows = kFlagIters * kTabThreads, kPassWords = kPassRows / 32;
  const int block_begin = blockIdx.x * rows_per_block;
  const int block_end = block_begin + rows_per_block < n_round ? block_begin + rows_per_block : n_round;
  for (int pass = block_begin; pass < block_end; pass += kPassRows) {
    const int begin = pass + wave * 64;
    float av[kFlagIters], as[kFlagIters];
#pragma unroll
    for (int it = 0; it < kFlagIters; ++it) {             // (n >= 1 here; what lies outside [n_sink, n) is masked below)
      const int i = begin + it * kTabThreads + lane, at = i < n ? i : n - 1;
      av[it] = ver[at];
      as[it] = sla[at];
    }
    if (pass == block_begin) {
      __builtin_amdgcn_sched_barrier(0);
      find_limits();
    }
#pragma unroll
    for (int it = 0; it < kFlagIters; ++it) {
      const int i = begin + it * kTabThreads + lane;
      const uint64_t in = __ballot(i >= s.n_sink) & __ballot(i < n);
      const uint64_t m0 = (__ballot(av[it] > tau_v) | __ballot(as[it] > tau_s)) & in;
      const uint64_t mm = (__ballot(av[it] > mean_v) | __ballot(as[it] > mean_s)) & in;
      if (lane == 0) {
        const int w = (it * kTabThreads + wave * 64) >> 5;
        w0[w] = (uint32_t)m0;
        w0[w + 1] = (uint32_t)(m0 >> 32);
        wm[w] = (uint32_t)mm;
        wm[w + 1] = (uint32_t)(mm >> 32);
      }
    }
    __syncthreads();
    {
      const int w = tid & (kPassWords - 1);
      const int gw = (pass >> 5) + w;
      if (gw < (n_round >> 5)) {
        if (tid < kPassWords) o0[gw] = w0[w];
        else if (tid < 2 * kPassWords) om[gw] = wm[w];
      }
    }
    __syncthreads();
  }
}

// Once the scale has become small it is folded into the stored values (A <- g A, g <- 1; the values g A
// do not change).  The head decides for itself from its own state, at the end of the update that
// made the scale small, so no host-side count is involved and a recorded graph folds when an eager run would.
// This step's additions may have been made in L2 (atomics): they are waited for, and the entries are then read
// with device-scope loads, which do not look at this CU's vector cache (it may hold the old values).
__device__ __forceinline__ void fold_scale(const Shape& s, int bh, double g1, float* ver, float* tab_sla, double* st,
                                           int tid, int threads) {
  if (g1 < kFoldBelow) {                                     // workgroup-uniform
    __threadfence();
    __syncthreads();
    float* sla_all = tab_sla + (int64_t)bh * 2 * s.Lcap;
    for (int i = tid; i < s.Lcap; i += threads) {
      const float x = __hip_atomic_load(&ver[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ver[i] = (float)(g1 * (double)x);
    }
    for (int i = tid; i < 2 * s.Lcap; i += threads) {
      const float x = __hip_atomic_load(&sla_all[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      sla_all[i] = (float)(g1 * (double)x);
    }
    __syncthreads();
    if (tid == 0) st[TS_G] = 1.0;
  }
}

// ----------------------------------------------------------------------------- update (Eq. 10)
// grid B*Hq.  The step saw n rows and selected idx[bh, 0:k_b] with scaled scores sc; entries outside
// [n_sink, n) are padding.  w = softmax over the valid entries; delta = w - 1/(2 * valid).
// kDistinct: the positions of a head's list are known to be distinct (the library's own Top-k, of more rows than
// k_table_update_own holds), so an entry's old value can be read beside the addition; otherwise (a caller's list, where a
// position may appear twice) every addition returns the value it found, which keeps the moments exact for a repeated
// position too.  256 heads, k = 6000: 107.5 us, 114.2 with additions that return.
template <bool kDistinct>
__global__ __launch_bounds__(kTabThreads) void k_table_update(Shape s, float* __restrict__ tab_ver,
                                                              float* __restrict__ tab_sla, double* __restrict__ state,
                                                              const int32_t* __restrict__ seq_lens,
                                                              const int32_t* __restrict__ idx,
                                                              const float* __restrict__ sc,
                                                              const int32_t* __restrict__ kk, double gamma,
                                                              const int32_t* __restrict__ gate,
                                                              int32_t* __restrict__ flags) {
  __shared__ double red[kTabThreads / 64];
  __shared__ float redf[kTabThreads / 64];
  const int bh = blockIdx.x, b = bh / s.Hq, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (gate && gate[bh] != 0) return;                        // bypassed head: Eq. 10 is skipped for it
  // The slash frame has room for Lcap - 1 moves since the tables were last written whole: past that the
  // update is refused here (the host refuses it too, but counts only the calls it sees, not graph replays).
  if (state[(int64_t)bh * kTableStateDoubles + TS_CNT] >= (double)(s.Lcap - 1)) {   // workgroup-uniform
    if (tid == 0) atomicOr(flags, LFPS_FLAG_TABLE_FULL);
    return;
  }
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  int kb = kk[b];
  kb = kb < 0 ? 0 : (kb > s.kmax ? s.kmax : kb);
  double* st = state + (int64_t)bh * kTableStateDoubles;
  const double g = st[TS_G];
  const int cnt = clamp_count(st[TS_CNT], s.Lcap);
  const int32_t* ih = idx + (int64_t)bh * s.kmax;
  const float* sh = sc + (int64_t)bh * s.kmax;
  float* ver = tab_ver + (int64_t)bh * s.Lcap;
  float* sla = tab_sla + (int64_t)bh * 2 * s.Lcap + (s.Lcap - cnt);   // indexed by position in the frame of this step

  // softmax over the valid selected entries
  float m = -INFINITY;
  int nvalid = 0;
  for (int e = tid; e < kb; e += kTabThreads) {
    const int p = ih[e];
    if (p >= s.n_sink && p < n) {
      m = fmaxf(m, sh[e]);
      ++nvalid;
    }
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) m = fmaxf(m, __shfl_xor(m, d));
  if (lane == 0) redf[wave] = m;
  __syncthreads();
  m = redf[0];
  for (int w = 1; w < kTabThreads / 64; ++w) m = fmaxf(m, redf[w]);
  double zsum = 0.0;
  for (int e = tid; e < kb; e += kTabThreads) {
    const int p = ih[e];
    if (p >= s.n_sink && p < n) zsum += (double)expf(sh[e] - m);
  }
  zsum = block_sum(zsum, red, tid);
  const double nv = block_sum((double)nvalid, red, tid);
  const double half = nv > 0.0 ? 0.5 / nv : 0.0;
  const double g1 = gamma * g;                               // scale after this step

  // selected entries: moments' change and the new unscaled values
  double dv[4] = {0, 0, 0, 0}, ds[4] = {0, 0, 0, 0};
  for (int e = tid; e < kb; e += kTabThreads) {
    const int p = ih[e];
    if (p >= s.n_sink && p < n) {
      const double delta = (double)expf(sh[e] - m) / zsum - half;
      const float inc = (float)(delta / g1);
      // (hardware fp32 adds in L2.)  Position p in the next frame (cnt + 1) is the slot of p - 1 in this one (for
      // p = 0 the never-written slot just below the frame).
      float old_v, old_s = 0.f;
      if constexpr (kDistinct) {
        old_v = ver[p];
        if (p - 1 >= s.n_sink) old_s = sla[p - 1];
        unsafeAtomicAdd(&ver[p], inc);
        unsafeAtomicAdd(&sla[p - 1], inc);
      } else {
        old_v = unsafeAtomicAdd(&ver[p], inc);
        old_s = unsafeAtomicAdd(&sla[p - 1], inc);
      }
      const double xv = gamma * g * (double)old_v;           // decayed old value
      const double xs = p - 1 >= s.n_sink ? gamma * g * (double)old_s : 0.0;   // decayed value moving in from p-1
      const double yv = xv + delta, ys = xs + delta;
      dv[0] += yv - xv;
      dv[1] += yv * yv - xv * xv;
      dv[2] += yv * yv * yv - xv * xv * xv;
      dv[3] += yv * yv * yv * yv - xv * xv * xv * xv;
      ds[0] += ys - xs;
      ds[1] += ys * ys - xs * xs;
      ds[2] += ys * ys * ys - xs * xs * xs;
      ds[3] += ys * ys * ys * ys - xs * xs * xs * xs;
    }
  }
  double tv[4], ts[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    tv[p] = block_sum(dv[p], red, tid);
    ts[p] = block_sum(ds[p], red, tid);
  }
  if (tid == 0) {
    double gp = 1.0;
    double Mv[4], Ms[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      gp *= gamma;
      Mv[p] = gp * st[TS_MV + p] + tv[p];
      Ms[p] = gp * st[TS_MS + p] + ts[p];
      st[TS_MV + p] = Mv[p];
      st[TS_MS + p] = Ms[p];
    }
    st[TS_G] = g1;
    st[TS_CNT] = (double)(cnt + 1);
    if (nv > 0.0) {                                          // entries were changed: no longer a flat table
      st[TS_FLAT_V] = 0.0;
      st[TS_FLAT_S] = 0.0;
    }
  }
  fold_scale(s, bh, g1, ver, tab_sla, st, tid, kTabThreads);
}

// The same for the library's own Top-k (distinct positions, at most kUpdateThreads * kUpdateEach of them): a thread reads
// its entries and the table values they change at once and keeps them, a plain store replaces the atomic addition, and
// the eight moments meet in one reduction.  The kernel is a chain of latencies (256 heads, k = 1024): 17.4 us with four
// entries per thread read three times and ten reductions one after the other, 8.2 us with eight sums each over all lanes of a
// wave, 6.7 us with the lanes sharing the sums out (wave_sum_of_8) and the old moments asked for at the start.
constexpr int kUpdateThreads = 1024, kUpdateEach = 4;

// The value of lane ^ 4 (DPP: lanes 4 to 7 and 12 to 15 from below, the others from above).
__device__ __forceinline__ double lane_xor4(double x) {
  auto half = [](int v) {
    const int t = __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xa, false);      // row_shr:4
    return __builtin_amdgcn_update_dpp(t, v, 0x104, 0xf, 0x5, false);             // row_shl:4
  };
  return __hiloint2double(half(__double2hiint(x)), half(__double2loint(x)));
}
__device__ __forceinline__ double lane_xor2(double x) {
  auto half = [](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, false); };      // quad_perm [2,3,0,1]
  return __hiloint2double(half(__double2hiint(x)), half(__double2loint(x)));
}
// Eight sums over a wave; lanes 2 p and 2 p + 1 of every sixteen return sum p.  Lanes 8, 4 and 2 apart share the values out while they
// add, so there are ten additions instead of 48, in the order of wave_sum.
__device__ __forceinline__ double wave_sum_of_8(const double (&d)[8], int lane) {
  double a[4], c[2];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const double keep = lane & 8 ? d[4 + p] : d[p], give = lane & 8 ? d[p] : d[4 + p];
    a[p] = keep + row16_rotate<8>(give);
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const double keep = lane & 4 ? a[2 + p] : a[p], give = lane & 4 ? a[p] : a[2 + p];
    c[p] = keep + lane_xor4(give);
  }
  const double keep = lane & 2 ? c[1] : c[0], give = lane & 2 ? c[0] : c[1];
  double v = keep + lane_xor2(give);
  auto swap = [](int x) { return __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, false); };      // quad_perm [1,0,3,2]
  v += __hiloint2double(swap(__double2hiint(v)), swap(__double2loint(v)));
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}

template <int kEach>
__global__ __launch_bounds__(kUpdateThreads) void k_table_update_own(Shape s, float* __restrict__ tab_ver,
                                                                     float* __restrict__ tab_sla,
                                                                     double* __restrict__ state,
                                                                     const int32_t* __restrict__ seq_lens,
                                                                     const int32_t* __restrict__ idx,
                                                                     const float* __restrict__ sc,
                                                                     const int32_t* __restrict__ kk, double gamma,
                                                                     const int32_t* __restrict__ gate,
                                                                     int32_t* __restrict__ flags) {
  request_arguments<decltype(&k_table_update_own<kEach>)>();
  constexpr int NT = kUpdateThreads, NW = NT / 64;
  __shared__ float top[NW];
  __shared__ double red[NW][8];
  __shared__ int cnts[NW];
  const int bh = blockIdx.x, b = bh / s.Hq, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int32_t* ih = idx + (int64_t)bh * s.kmax;
  const float* sh = sc + (int64_t)bh * s.kmax;
  int pos[kEach];
  float x[kEach];
#pragma unroll
  for (int u = 0; u < kEach; ++u) {                          // (up to the row length; masked below)
    const int e = tid + u * NT;
    pos[u] = e < s.kmax ? ih[e] : -1;
    x[u] = e < s.kmax ? sh[e] : 0.f;
  }
  double* st = state + (int64_t)bh * kTableStateDoubles;
  const double g = st[TS_G], moves = st[TS_CNT];
  const int at_moment = (tid & 4 ? TS_MS : TS_MV) + (tid & 3);
  const double old_moment = st[at_moment];                   // (of threads 0 to 7)
  int n = seq_lens[b];
  int kb = kk[b];
  if (gate && gate[bh] != 0) return;                        // bypassed head: Eq. 10 is skipped for it
  if (moves >= (double)(s.Lcap - 1)) {                       // no room in the slash frame (see k_table_update)
    if (tid == 0) atomicOr(flags, LFPS_FLAG_TABLE_FULL);
    return;
  }
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  kb = kb < 0 ? 0 : (kb > s.kmax ? s.kmax : kb);
  const int cnt = clamp_count(moves, s.Lcap);
  float* ver = tab_ver + (int64_t)bh * s.Lcap;
  float* sla = tab_sla + (int64_t)bh * 2 * s.Lcap + (s.Lcap - cnt);   // indexed by position in the frame of this step
  bool ok[kEach];
  float old_v[kEach], old_s[kEach];
  float m = -INFINITY;
  int valid = 0;
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    ok[u] = tid + u * NT < kb && pos[u] >= s.n_sink && pos[u] < n;
    // position p in the next frame (cnt + 1) is the slot of p - 1 in this one (p = 0: the slot just below the frame)
    old_v[u] = ok[u] ? ver[pos[u]] : 0.f;
    old_s[u] = ok[u] ? sla[pos[u] - 1] : 0.f;
    m = ok[u] ? fmaxf(m, x[u]) : m;
    valid += __popcll(__ballot(ok[u]));
  }
  m = row16_max(m);
  m = fmaxf(m, __shfl_xor(m, 16));
  m = fmaxf(m, __shfl_xor(m, 32));
  if (lane == 0) {
    top[wave] = m;
    cnts[wave] = valid;
  }
  __syncthreads();
  m = top[0];
  valid = cnts[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) {
    m = fmaxf(m, top[w]);
    valid += cnts[w];
  }
  auto wave_sum = [](double v) {
    v = row16_sum(v);
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    return v;
  };
  float w_[kEach];
  double zsum = 0.0;
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    w_[u] = ok[u] ? expf(x[u] - m) : 0.f;
    zsum += (double)w_[u];
  }
  zsum = wave_sum(zsum);
  if (lane == 0) red[wave][0] = zsum;
  __syncthreads();
  zsum = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) zsum += red[w][0];
  const double half = valid > 0 ? 0.5 / (double)valid : 0.0;
  const double g1 = gamma * g;                               // scale after this step
  double d[8] = {0, 0, 0, 0, 0, 0, 0, 0};                    // change of the moments: vertical, slash
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    if (ok[u]) {
      const double delta = (double)w_[u] / zsum - half;
      const float inc = (float)(delta / g1);
      ver[pos[u]] = old_v[u] + inc;
      sla[pos[u] - 1] = old_s[u] + inc;
      const double xv = g1 * (double)old_v[u];                                     // decayed old value
      const double xs = pos[u] - 1 >= s.n_sink ? g1 * (double)old_s[u] : 0.0;      // decayed value moving in from p - 1
      double yv = xv + delta, ys = xs + delta, av = xv, as = xs;
      const double bv = yv, bs = ys;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        d[p] += yv - av;
        d[4 + p] += ys - as;
        yv *= bv;
        ys *= bs;
        av *= xv;
        as *= xs;
      }
    }
  }
  const double moment = wave_sum_of_8(d, lane);
  __syncthreads();                                           // everybody has read red[][0]
  if (lane < 16 && !(lane & 1)) red[wave][lane >> 1] = moment;
  __syncthreads();
  if (tid < 8) {                                             // thread p: moment p & 3 of the vertical, then of the slash table
    double sum = 0.0, gp = 1.0;
    for (int w = 0; w < NW; ++w) sum += red[w][tid];
    for (int p = 0; p <= (tid & 3); ++p) gp *= gamma;
    st[at_moment] = gp * old_moment + sum;
    if (tid == 0) {
      st[TS_G] = g1;
      st[TS_CNT] = (double)(cnt + 1);
      if (valid > 0) {                                       // entries were changed: no longer a flat table
        st[TS_FLAT_V] = 0.0;
        st[TS_FLAT_S] = 0.0;
      }
    }
  }
  fold_scale(s, bh, g1, ver, tab_sla, st, tid, NT);
}

// ----------------------------------------------------------------------------- import / export / renormalise
// Import true table values phi_*[bh, 0:n_b] (fp32, position frame): scale 1, count 0, dense moments.
__global__ __launch_bounds__(kTabThreads) void k_table_import(Shape s, float* __restrict__ tab_ver,
                                                              float* __restrict__ tab_sla, double* __restrict__ state,
                                                              const int32_t* __restrict__ seq_lens,
                                                              const float* __restrict__ phi_ver,
                                                              const float* __restrict__ phi_sla) {
  __shared__ double red[kTabThreads / 64];
  __shared__ float redf[kTabThreads / 64];
  const int bh = blockIdx.x, b = bh / s.Hq, tid = threadIdx.x;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  float* ver = tab_ver + (int64_t)bh * s.Lcap;
  float* sla = tab_sla + (int64_t)bh * 2 * s.Lcap;
  const float* pv = phi_ver + (int64_t)bh * s.Lcap;
  const float* ps = phi_sla + (int64_t)bh * s.Lcap;
  double mv[4] = {0, 0, 0, 0}, ms[4] = {0, 0, 0, 0};
  float lo_v = INFINITY, hi_v = -INFINITY, lo_s = INFINITY, hi_s = -INFINITY;
  for (int i = tid; i < 2 * s.Lcap; i += kTabThreads) sla[i] = 0.f;
  __syncthreads();
  for (int i = tid; i < s.Lcap; i += kTabThreads) {
    const bool in = i >= s.n_sink && i < n;
    const float xv = in ? pv[i] : 0.f, xs = in ? ps[i] : 0.f;
    ver[i] = xv;
    sla[i + s.Lcap] = xs;
    if (in) {
      const double a1 = xv, b1 = xs;
      mv[0] += a1; mv[1] += a1 * a1; mv[2] += a1 * a1 * a1; mv[3] += a1 * a1 * a1 * a1;
      ms[0] += b1; ms[1] += b1 * b1; ms[2] += b1 * b1 * b1; ms[3] += b1 * b1 * b1 * b1;
      lo_v = fminf(lo_v, xv); hi_v = fmaxf(hi_v, xv);
      lo_s = fminf(lo_s, xs); hi_s = fmaxf(hi_s, xs);
    }
  }
  double Mv[4], Ms[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    Mv[p] = block_sum(mv[p], red, tid);
    Ms[p] = block_sum(ms[p], red, tid);
  }
  // a flat table (every entry equal) has no pattern: block minimum == block maximum
  lo_v = block_min(lo_v, redf, tid);
  hi_v = -block_min(-hi_v, redf, tid);
  lo_s = block_min(lo_s, redf, tid);
  hi_s = -block_min(-hi_s, redf, tid);
  const double N = (double)(n - s.n_sink > 0 ? n - s.n_sink : 0);
  if (tid == 0) {
    double* st = state + (int64_t)bh * kTableStateDoubles;
    st[TS_G] = 1.0;
    st[TS_CNT] = 0.0;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      st[TS_MV + p] = Mv[p];
      st[TS_MS + p] = Ms[p];
    }
    st[TS_FLAT_V] = hi_v > lo_v ? 0.0 : 1.0;
    st[TS_FLAT_S] = hi_s > lo_s ? 0.0 : 1.0;
    st[TS_FLAT_N] = N;
  }
}

// True table values of positions [0, n_b) as fp64 (zeros elsewhere up to Lcap).
__global__ __launch_bounds__(kTabThreads) void k_table_export(Shape s, const float* __restrict__ tab_ver,
                                                              const float* __restrict__ tab_sla,
                                                              const double* __restrict__ state,
                                                              const int32_t* __restrict__ seq_lens,
                                                              double* __restrict__ phi_ver,
                                                              double* __restrict__ phi_sla) {
  const int bh = blockIdx.y, b = bh / s.Hq;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const double* st = state + (int64_t)bh * kTableStateDoubles;
  const double g = st[TS_G];
  const int cnt = clamp_count(st[TS_CNT], s.Lcap);
  const int i = blockIdx.x * kTabThreads + threadIdx.x;
  if (i >= s.Lcap) return;
  const bool in = i >= s.n_sink && i < n;
  phi_ver[(int64_t)bh * s.Lcap + i] = in ? g * (double)tab_ver[(int64_t)bh * s.Lcap + i] : 0.0;
  phi_sla[(int64_t)bh * s.Lcap + i] = in ? g * (double)tab_sla[(int64_t)bh * 2 * s.Lcap + (s.Lcap - cnt) + i] : 0.0;
}

// ----------------------------------------------------------------------------- Eq. 4
// Tables from the attention weights of the last s prefill queries.  One launch per query: the j-th most
// recent query (j = 1..s) sees rows [0, n_b - j + 1); its weights w (softmax over the offloaded rows it
// sees) are added to the vertical table at i and to the slash table at i + j - 1 (Eq. 4's w_{i-j+1}),
// times 1/(2 s (1 - gamma)).  j = 1 overwrites, later launches accumulate.  score[bh, 0:n_b] holds the
// scaled scores of query j.  grid B*Hq.  launch_table_state then derives the statistics.
// Used for fp32 caches; the other formats take all queries together (prefill.hip).
__global__ __launch_bounds__(1024) void k_table_init(Shape s, float* __restrict__ tab_ver, float* __restrict__ tab_sla,
                                                     const int32_t* __restrict__ seq_lens,
                                                     const float* __restrict__ score, int64_t score_stride, double gamma,
                                                     int j, int n_queries) {
  __shared__ double red[16];
  __shared__ float redf[16];
  const int bh = blockIdx.x, b = bh / s.Hq, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const int seen = n - j + 1 > 0 ? n - j + 1 : 0;           // rows query j sees
  const float* sc = score + (int64_t)bh * score_stride;
  float* ver = tab_ver + (int64_t)bh * s.Lcap;
  float* sla = tab_sla + (int64_t)bh * 2 * s.Lcap + s.Lcap;  // position frame (update count 0)
  float m = -INFINITY;
  for (int i = s.n_sink + tid; i < seen; i += 1024) m = fmaxf(m, sc[i]);
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) m = fmaxf(m, __shfl_xor(m, d));
  if (lane == 0) redf[wave] = m;
  __syncthreads();
  m = redf[0];
  for (int w = 1; w < 16; ++w) m = fmaxf(m, redf[w]);
  double z = 0.0;
  for (int i = s.n_sink + tid; i < seen; i += 1024) z += (double)expf(sc[i] - m);
  z = block_sum(z, red, tid);
  const double norm = z > 0.0 ? 1.0 / (2.0 * (double)n_queries * (1.0 - gamma) * z) : 0.0;
  if (j == 1) {
    for (int i = tid; i < s.Lcap; i += 1024) {
      ver[i] = 0.f;
      sla[i - s.Lcap] = 0.f;
      sla[i] = 0.f;
    }
    __syncthreads();
  }
  // a position receives at most one vertical and one slash contribution per launch: plain read-modify-write
  for (int i = s.n_sink + tid; i < seen; i += 1024) {
    const float x = (float)((double)expf(sc[i] - m) * norm);
    ver[i] += x;
    sla[i + j - 1] += x;                                     // i + j - 1 <= n - 1
  }
}

// ----------------------------------------------------------------------------- head sparsity (Eq. 5, Eq. 6)
// One wave per (b, h), a chain of latencies: a row at a time, 64 lanes wide, took 10.6 us at 256 heads and 10 rows; four rows
// side by side and all of them requested at once, 5.4 us; with one fp64 exponential for both sets and one logarithm for the
// three, in neighbouring lanes, 5.2 (sixteen table steps 1078 -> 1073 us in all).  rho = w_sink / (w_sink + w_global + w_local):
//   w_sink   = sum over rows [0, n_sink) of exp(q.K_i/sqrt(D)),
//   w_global = n * exp(q.kbar/sqrt(D) + |q|^2 sigma2_hat / 2)        (log-normal mean of the weights, App. B.1),
//   w_local  = sum over the newest n_local rows of exp(q.K_i/sqrt(D)).
// A head with rho > eps is bypassed: its output row is vbar, its index row -1 (Alg. 1 lines 1-4); the later
// kernels of the step skip it.  The three terms are kept as exponent + log-sum so that a dominant sink
// (logit in the hundreds) cannot overflow.
template <typename T, bool kPaged>
__global__ __launch_bounds__(64) void k_head_sparsity(Shape s, const float* __restrict__ q, const T* __restrict__ K,
                                                      int64_t stride_b, int64_t stride_h, int64_t stride_n, KvPage pg,
                                                      const int32_t* __restrict__ seq_lens,
                                                      const float* __restrict__ kbar,
                                                      const float* __restrict__ sigma2_hat, int n_local, float eps,
                                                      float* __restrict__ rho_out, int32_t* __restrict__ gate_out,
                                                      const float* __restrict__ vbar, int32_t* __restrict__ topk_idx,
                                                      float* __restrict__ topk_score, float* __restrict__ out) {
  request_arguments<decltype(&k_head_sparsity<T, kPaged>)>();
  const int bh = blockIdx.x, b = bh / s.Hq, h = bh % s.Hq, g = h / s.G, lane = threadIdx.x;
  const int j = lane & 15, rs = lane >> 4;                    // 16 lanes per row, 8 channels each
  int n = seq_lens[b];
  n = n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n);
  const float scale = 0.08838834764831845f;
  float qr[8], kr[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {                               // (a caller's pointers: no more than 4-byte alignment)
    qr[c] = q[(int64_t)bh * kD + 8 * j + c];
    kr[c] = kbar[((int64_t)b * s.Hkv + g) * kD + 8 * j + c];
  }
  using Rows = RowMap<kPaged>;
  const T* Kbg = K + Rows::base(b, g, stride_b, stride_h) + 8 * j;
  const int ns = s.n_sink < n ? s.n_sink : n;
  const int lo = n - n_local > 0 ? n - n_local : 0;
  const int rows = ns + (n - lo);                             // the sinks, then the newest rows
  // log-sum-exp of both sets, sixteen rows at a time: four per lane group, all loads issued together; then lane i of a
  // group takes row i (a logit is an fp32 number, its exponential and the sums are fp64)
  double m_sink = -INFINITY, z_sink = 0.0, m_loc = -INFINITY, z_loc = 0.0;
  for (int r0 = 0; r0 < rows; r0 += 16) {
    int prow[4];
    Raw8<T> raw[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = r0 + 4 * u + rs < rows ? r0 + 4 * u + rs : rows - 1;
      prow[u] = Rows::phys(pg, b, r < ns ? r : lo + r - ns);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) raw[u].load(Kbg + Rows::offset(pg, prow[u], stride_b, stride_n));
    float mine = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float x[8];
      raw[u].get(x);
      float d = 0.f;
#pragma unroll
      for (int c = 0; c < 8; ++c) d = fmaf(qr[c], x[c], d);
      d = row16_sum(d) * scale;
      const float of_row = __shfl(d, 16 * (j & 3));           // rows r0 + 4 u + (j & 3)
      mine = (j >> 2) == u ? of_row : mine;
    }
    // both sets in one exponential: a row is in one of them
    const int r = r0 + j;
    const bool sink = r < ns, local = r >= ns && r < rows;
    const float top_sink = row16_max(sink ? mine : -INFINITY), top_loc = row16_max(local ? mine : -INFINITY);
    const double mx_sink = m_sink > (double)top_sink ? m_sink : (double)top_sink;
    const double mx_loc = m_loc > (double)top_loc ? m_loc : (double)top_loc;
    const double mx = sink ? mx_sink : mx_loc;
    // (a logit of +inf is a term of weight 1 beside which all others vanish; a NaN stays)
    const double term = sink || local ? ((double)mine == mx ? 1.0 : exp((double)mine - mx)) : 0.0;
    auto add = [&](float top, bool in, double to, double& m, double& z) {
      const double part = row16_sum(in ? term : 0.0);
      if (top == -INFINITY) return;                            // (wave-uniform: every group holds the same rows)
      if (r0 > 0) z = m == to ? z : z * exp(m - to);           // (nothing before the first rows)
      z += part;
      m = to;
    };
    add(top_sink, sink, mx_sink, m_sink, z_sink);
    add(top_loc, local, mx_loc, m_loc, z_loc);
  }
  float dk = 0.f, qq = 0.f;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    dk = fmaf(qr[c], kr[c], dk);
    qq = fmaf(qr[c], qr[c], qq);
  }
  dk = row16_sum(dk);
  qq = row16_sum(qq);
  // the three logarithms, and then the two exponentials, by neighbouring lanes at once
  const double ln = log(j == 0 ? (double)n : (j == 1 ? z_sink : z_loc));
  const double l_glob = n > 0 ? __shfl(ln, 0) + (double)(dk * scale) + (double)qq * (double)sigma2_hat[bh] * 0.5 : -INFINITY;
  const double l_sink = z_sink > 0.0 ? m_sink + __shfl(ln, 1) : -INFINITY;
  const double l_loc = z_loc > 0.0 ? m_loc + __shfl(ln, 2) : -INFINITY;
  // rho = exp(l_sink) / (exp(l_sink) + exp(l_glob) + exp(l_loc))
  double rho = 0.0;
  if (l_sink > -INFINITY) {                                     // (uniform)
    const double e = exp((j == 0 ? l_glob : l_loc) - l_sink);
    rho = 1.0 / (1.0 + __shfl(e, 0) + __shfl(e, 1));
  }
  const bool bypass = rho > (double)eps;
  if (lane == 0) {
    if (rho_out) rho_out[bh] = (float)rho;
    gate_out[bh] = bypass ? 1 : 0;
  }
  if (bypass && out) {
    out[(int64_t)bh * kD + 2 * lane] = vbar[((int64_t)b * s.Hkv + g) * kD + 2 * lane];
    out[(int64_t)bh * kD + 2 * lane + 1] = vbar[((int64_t)b * s.Hkv + g) * kD + 2 * lane + 1];
    for (int i = lane; i < s.kmax; i += 64) {
      topk_idx[(int64_t)bh * s.kmax + i] = -1;
      if (topk_score) topk_score[(int64_t)bh * s.kmax + i] = 0.f;
    }
  }
}

// ----------------------------------------------------------------------------- launchers
hipError_t launch_table_flags(const Shape& s, const float* tab_ver, const float* tab_sla, const double* state,
                              const int32_t* seq_lens, uint32_t* f0, uint32_t* fm, int flag_words, double a,
                              const int32_t* gate, hipStream_t st) {
  // about 4096 workgroups in all, each a whole number of passes
  const int pass_rows = kTabThreads * kFlagIters;
  int per_head = 4096 / (s.B * s.Hq);
  per_head = per_head < 1 ? 1 : per_head;
  int rows_per_block = ((s.Lcap + per_head - 1) / per_head + pass_rows - 1) / pass_rows * pass_rows;
  if (rows_per_block < pass_rows) rows_per_block = pass_rows;
  const int chunks = (s.Lcap + rows_per_block - 1) / rows_per_block;
  hipLaunchKernelGGL(k_table_flags, dim3(chunks, s.B * s.Hq), dim3(kTabThreads), 0, st, s, tab_ver, tab_sla, state,
                     seq_lens, f0, fm, flag_words, rows_per_block, a, gate);
  return hipGetLastError();
}

hipError_t launch_table_update(const Shape& s, float* tab_ver, float* tab_sla, double* state, const int32_t* seq_lens,
                               const int32_t* idx, const float* sc, const int32_t* k, double gamma, const int32_t* gate,
                               int32_t* flags, bool distinct, hipStream_t st) {
#define LFPS_UPDATE(KERNEL, THREADS)                                                                               \
  hipLaunchKernelGGL((KERNEL), dim3(s.B * s.Hq), dim3(THREADS), 0, st, s, tab_ver, tab_sla, state, seq_lens, idx, sc, \
                     k, gamma, gate, flags)
  if (!distinct) LFPS_UPDATE(k_table_update<false>, kTabThreads);
  else if (s.kmax > kUpdateThreads * kUpdateEach) LFPS_UPDATE(k_table_update<true>, kTabThreads);
  else if (s.kmax > kUpdateThreads) LFPS_UPDATE(k_table_update_own<kUpdateEach>, kUpdateThreads);
  else LFPS_UPDATE(k_table_update_own<1>, kUpdateThreads);
#undef LFPS_UPDATE
  return hipGetLastError();
}

hipError_t launch_table_import(const Shape& s, float* tab_ver, float* tab_sla, double* state, const int32_t* seq_lens,
                               const float* phi_ver, const float* phi_sla, hipStream_t st) {
  hipLaunchKernelGGL(k_table_import, dim3(s.B * s.Hq), dim3(kTabThreads), 0, st, s, tab_ver, tab_sla, state, seq_lens,
                     phi_ver, phi_sla);
  return hipGetLastError();
}

hipError_t launch_table_export(const Shape& s, const float* tab_ver, const float* tab_sla, const double* state,
                               const int32_t* seq_lens, double* phi_ver, double* phi_sla, hipStream_t st) {
  hipLaunchKernelGGL(k_table_export, dim3((s.Lcap + kTabThreads - 1) / kTabThreads, s.B * s.Hq), dim3(kTabThreads), 0,
                     st, s, tab_ver, tab_sla, state, seq_lens, phi_ver, phi_sla);
  return hipGetLastError();
}

hipError_t launch_table_init(const Shape& s, float* tab_ver, float* tab_sla, const int32_t* seq_lens,
                             const float* score, int64_t score_stride, double gamma, int j, int n_queries,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_table_init, dim3(s.B * s.Hq), dim3(1024), 0, st, s, tab_ver, tab_sla, seq_lens, score,
                     score_stride, gamma, j, n_queries);
  return hipGetLastError();
}

hipError_t launch_head_sparsity(const Shape& s, int dtype, const float* q, const KvView& kv, const float* kbar,
                                const float* sigma2_hat, int n_local, float eps, float* rho, int32_t* gate,
                                const float* vbar, int32_t* topk_idx, float* topk_score, float* out, hipStream_t st) {
#define LFPS_LAUNCH_HSP(TYPE, PAGED)                                                                             \
  hipLaunchKernelGGL((k_head_sparsity<TYPE, PAGED>), dim3(s.B * s.Hq), dim3(64), 0, st, s, q, (const TYPE*)kv.k,     \
                     kv.stride_b, kv.stride_h, kv.stride_n, kv.page, kv.seq_lens, kbar, sigma2_hat, n_local, eps, rho, \
                     gate, vbar, topk_idx, topk_score, out)
  const bool paged = kv.page.table != nullptr;
  if (dtype == LFPS_BF16 && kv.k_fp8) {
    if (paged) LFPS_LAUNCH_HSP(uint8_t, true);
    else LFPS_LAUNCH_HSP(uint8_t, false);
  } else if (dtype == LFPS_BF16) {
    if (paged) LFPS_LAUNCH_HSP(uint16_t, true);
    else LFPS_LAUNCH_HSP(uint16_t, false);
  } else if (dtype == LFPS_F16) {
    if (paged) LFPS_LAUNCH_HSP(_Float16, true);
    else LFPS_LAUNCH_HSP(_Float16, false);
  } else {
    if (paged) LFPS_LAUNCH_HSP(float, true);
    else LFPS_LAUNCH_HSP(float, false);
  }
#undef LFPS_LAUNCH_HSP
  return hipGetLastError();
}

}  // namespace lfps
