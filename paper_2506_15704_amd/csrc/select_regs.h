// The select for heads whose scored rows fit the registers of one workgroup (up to kRegElems per thread): every element
// is read once and stays in a register through all passes, so a pass costs no memory traffic and the select is a short
// chain of LDS round trips (select_body.h keeps the rows in LDS or streams them, for longer lists).
#pragma once
#include <type_traits>

#include "select_body.h"

namespace lfps {

constexpr int kRegElems = 16;

// A selected row as the attention reads it: physical row and softmax numerator (a row to skip: the request's row 0,
// weight 0).
struct SelRow {
  int32_t row;
  float p;
};

// Histogram bin of score x for a lower bound lo of all scores: 64 bins per octave of x - lo + 1/16, so bins are 1/1024
// wide at the bound and grow with the distance.  Survivors of a threshold pile up just above it, where the k-th best
// lies; scores far above share wide bins.  Monotone in x, whatever x and lo are.
__device__ __forceinline__ int tail_bin(float x, float lo, int bins) {
  const float t = fmaxf(x - lo, 0.f) + 0.0625f;
  const int b = (int)((__float_as_uint(t) - 0x3D800000u) >> 17);
  return b < bins ? b : bins - 1;
}

// The ksel best of the workgroup's n elements (1 <= ksel <= n): thread t holds the elements u*NT + t (score v[u],
// sanitised), which ascend in position over u and then t: a wave's loads, and its stores of selected elements, touch
// consecutive entries.  lo: a lower bound of all scores, or (from_min) ignored and
// replaced by their minimum.  All threads call, after a barrier behind sm.hist = 0 and sm.list_n = 0.  Calls
// out(rank, u, top) for every selected element, rank = its place in ascending position, top = the largest score; equal
// scores at the cut go to the lower position.  *thr_out receives the ksel-th best score.
// kScalarMax: a wave's largest and smallest score pass through a scalar register, see k_filter_select_attend.
template <int NT, int E, bool kScalarMax = false, typename Out>
__device__ __forceinline__ void select_registers(SelectShared<NT>& sm, const float (&v)[E], int n, int ksel, float lo,
                                                 bool from_min, float* __restrict__ thr_out, Out out) {
  constexpr int kWaves = NT / 64, kBins = 2 * NT, kListCap = NT;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  static_assert(kWaves <= 16, "the waves' values are merged in a row of lanes");
  auto mine = [&](int u) { return u * NT + tid < n; };
  float hi = -FLT_MAX, mn = FLT_MAX;
#pragma unroll
  for (int u = 0; u < E; ++u) {
    hi = mine(u) ? fmaxf(hi, v[u]) : hi;
    mn = mine(u) ? fminf(mn, v[u]) : mn;
  }
  constexpr int kLeader = kScalarMax ? 0 : 63;             // stores for the wave
  auto settled = [](float x) { return kScalarMax ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63)) : x; };
  hi = settled(wave_max_in_last(hi));
  if (lane == kLeader) sm.whi[wv] = hi;
  if (from_min) {
    mn = -settled(wave_max_in_last(-mn));
    if (lane == kLeader) sm.wlo[wv] = mn;
    __syncthreads();
    lo = -__int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(row16_max(lane < kWaves ? -sm.wlo[lane] : -FLT_MAX))));
  }
  // (bins are computed where they are needed: held for all elements they would cost E registers)
#pragma unroll
  for (int u = 0; u < E; ++u)
    if (mine(u)) atomicAdd(&sm.hist[tail_bin(v[u], lo, kBins)], 1u);
  __syncthreads();
  const float top = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(row16_max(lane < kWaves ? sm.whi[lane] : -FLT_MAX))));
  find_bin(sm, (uint32_t)ksel, tid, lane, wv);
  const int tb = (int)sm.bin;
  uint32_t need = sm.need;                                 // elements still to take from bin tb (>= 1)
  const uint32_t m = sm.hist[tb];
  uint32_t thr_key, need_eq;
  if (m <= (uint32_t)kListCap) {
#pragma unroll
    for (int u = 0; u < E; ++u) {
      const bool hit = mine(u) && tail_bin(v[u], lo, kBins) == tb;
      const uint64_t mh = __ballot(hit);
      if (mh) {
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&sm.list_n, (uint32_t)__popcll(mh));
        at = (uint32_t)__builtin_amdgcn_readlane((int)at, 0);
        if (hit) sm.list[at + lanes_below(mh)] = f2key(v[u]);
      }
    }
    __syncthreads();
    // few members (the usual case): every wave ranks them by itself and no further barrier is needed
    const bool few = m <= 64u;
    const uint32_t cand = few ? (uint32_t)lane : (uint32_t)tid;
    const uint32_t key = cand < m ? sm.list[cand] : 0u;
    uint32_t gt = 0, ge = 0;
    for (uint32_t i = 0; i < m; ++i) {
      const uint32_t o = sm.list[i];
      gt += o > key;
      ge += o >= key;
    }
    const bool is_thr = cand < m && gt < need && need <= ge;       // (equal keys agree)
    if (few) {
      const int src = __builtin_ctzll(__ballot(is_thr));
      thr_key = (uint32_t)__builtin_amdgcn_readlane((int)key, src);
      need_eq = need - (uint32_t)__builtin_amdgcn_readlane((int)gt, src);
    } else {
      if (is_thr) {
        sm.thr = key;
        sm.need_eq = need - gt;
      }
      __syncthreads();
      thr_key = sm.thr;
      need_eq = sm.need_eq;
    }
  } else {                                                 // a crowded bin: radix descent over the members' keys
    uint32_t prefix = 0, mask = 0;
#pragma unroll 1
    for (int pass = 0; pass < 4; ++pass) {
      const int shift = pass < 3 ? 32 - 9 * (pass + 1) : 0;
      const uint32_t dmask = pass < 3 ? 511u : 31u;
      __syncthreads();
      for (int i = tid; i < kBins; i += NT) sm.hist[i] = 0u;
      __syncthreads();
#pragma unroll
      for (int u = 0; u < E; ++u) {
        const uint32_t key = f2key(v[u]);
        if (mine(u) && tail_bin(v[u], lo, kBins) == tb && ((key ^ prefix) & mask) == 0u)
          atomicAdd(&sm.hist[(key >> shift) & dmask], 1u);
      }
      __syncthreads();
      find_bin(sm, need, tid, lane, wv);
      prefix |= sm.bin << shift;
      need = sm.need;
      mask |= dmask << shift;
    }
    thr_key = prefix;
    need_eq = need;
  }
  const float thr = key2f(thr_key);
  if (thr_out && tid == 0) *thr_out = thr;
  // ordered compaction: everything above the threshold, and the first need_eq elements equal to it.  Per 64 elements
  // (u, wave) the counts go to LDS (elements > thr) << 16 | (elements == thr); every wave scans all of them.
  uint32_t* counts = sm.hist;                              // (not read any more)
#pragma unroll
  for (int u = 0; u < E; ++u) {
    const uint32_t gt = __popcll(__ballot(mine(u) && v[u] > thr)), eq = __popcll(__ballot(mine(u) && v[u] == thr));
    if (lane == 0) counts[u * kWaves + wv] = gt << 16 | eq;
  }
  __syncthreads();
  constexpr int kRows = (E * kWaves + 63) / 64;
  uint32_t before[kRows];                                  // exclusive prefix of entry 64 i + lane
  uint32_t carry = 0;
#pragma unroll
  for (int i = 0; i < kRows; ++i) {
    const uint32_t x = 64 * i + lane < E * kWaves ? counts[64 * i + lane] : 0u;
    const uint32_t inc = (uint32_t)wave_inclusive_sum((int)x);
    before[i] = carry + inc - x;
    carry += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
  }
#pragma unroll
  for (int u = 0; u < E; ++u) {
    const uint64_t gt = __ballot(mine(u) && v[u] > thr), eq = __ballot(mine(u) && v[u] == thr);
    if (!(gt | eq)) continue;
    const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)before[u * kWaves / 64], (u * kWaves) % 64 + wv);
    const uint32_t eq_before = (at & 0xFFFFu) + lanes_below(eq);
    const bool take = mine(u) && (v[u] > thr || (v[u] == thr && eq_before < need_eq));
    const uint32_t rank = (at >> 16) + lanes_below(gt) + (eq_before < need_eq ? eq_before : need_eq);
    if (take && rank < (uint32_t)ksel) out((int)rank, u, top);
  }
}

// The select above on kept (score, element) pairs in LDS, ascending in position, all of them >= cut: out(rank, element, score).
// All threads call, after a barrier behind the list's last entry.
template <int NT, typename Out>
__device__ __forceinline__ void select_list(SelectShared<NT>& sm, const float2* list, int kept, int ksel, float cut,
                                            float* __restrict__ thr_out, Out out) {
  for (int i = threadIdx.x; i < 2 * NT; i += NT) sm.hist[i] = 0u;
  if (threadIdx.x == 0) sm.list_n = 0u;
  __syncthreads();
  auto finish = [&](auto elems) {
    constexpr int E2 = decltype(elems)::value;
    float w[E2];
    int at[E2];
#pragma unroll
    for (int u = 0; u < E2; ++u) {
      const int e = u * NT + (int)threadIdx.x < kept ? u * NT + (int)threadIdx.x : kept - 1;
      w[u] = list[e].x;
      at[u] = __float_as_int(list[e].y);
    }
    select_registers<NT, E2>(sm, w, kept, ksel, cut, false, thr_out,
                             [&](int rank, int u, float) { out(rank, at[u], w[u]); });
  };
  if (kept <= 2 * NT) finish(std::integral_constant<int, 2>{});
  else if (kept <= 4 * NT) finish(std::integral_constant<int, 4>{});
  else finish(std::integral_constant<int, kRegElems>{});
}

// The same for a row whose scoring pass has left the largest (sanitised) score of every 16 in tops[0 .. (n + 15) / 16 - 1],
// at least ksel and at most kRegElems * NT of them.  The ksel best of these, ties to the lower block, tell the blocks
// that hold the ksel best scores: ksel scores reach the smallest of them, t, so no smaller one is taken; every block with a
// larger score is among them; and of scores equal to t the first ones are, because the last block chosen for a top equal to
// t leaves enough of them before it.  What reaches t in those blocks goes to LDS, ascending, and is selected from there.
// Bound by the latency of one CU; 32 heads x 32768 scores, k = 1024: 15.5 us, 25 with select_long, which handles every score
// four times.  False if more than cap elements would go to the list: nothing has been written then.  sc: 16-byte aligned, readable up to
// a multiple of 16.
template <int NT, typename Out>
__device__ __forceinline__ bool select_blocks(SelectShared<NT>& sm, const float* __restrict__ sc,
                                              const float* __restrict__ tops, int n, int ksel, float2* list, int cap,
                                              float* __restrict__ thr_out, Out out) {
  constexpr int kWaves = NT / 64;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int nb = (n + 15) >> 4;
  cap -= (ksel + 1) >> 1;                                  // the chosen blocks lie behind the list
  uint32_t* blocks = reinterpret_cast<uint32_t*>(list + cap);
  for (int i = tid; i < 2 * NT; i += NT) sm.hist[i] = 0u;
  if (tid == 0) sm.list_n = 0u;
  __syncthreads();
  auto choose = [&](auto elems) {
    constexpr int E = decltype(elems)::value;
    float v[E];
#pragma unroll
    for (int u = 0; u < E; ++u) v[u] = tops[u * NT + tid < nb ? u * NT + tid : nb - 1];
    select_registers<NT, E>(sm, v, nb, ksel, 0.f, true, &sm.cut,
                            [&](int rank, int u, float) { blocks[rank] = (uint32_t)(u * NT + tid); });
  };
  if (nb <= 2 * NT) choose(std::integral_constant<int, 2>{});
  else if (nb <= 4 * NT) choose(std::integral_constant<int, 4>{});
  else if (nb <= 8 * NT) choose(std::integral_constant<int, 8>{});
  else choose(std::integral_constant<int, kRegElems>{});
  __syncthreads();
  const float cut = sm.cut;
  int kept = 0;
#pragma unroll 1
  for (int r0 = 0; r0 < ksel; r0 += NT) {                  // a block a thread
    const bool in = r0 + tid < ksel;
    const int base = in ? (int)blocks[r0 + tid] << 4 : 0;
    float x[16];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const f32x4 y = reinterpret_cast<const f32x4*>(sc + base)[c];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[4 * c + i] = y[i];
    }
    uint32_t take = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      x[i] = sanitize(x[i]);
      take |= (in && base + i < n && x[i] >= cut ? 1u : 0u) << i;
    }
    const int cnt = __popc(take), inc = wave_inclusive_sum(cnt);
    if (lane == 63) sm.wsum[wv] = (uint32_t)inc;
    __syncthreads();
    int at = kept + inc - cnt, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int t = (int)sm.wsum[w];
      at += w < wv ? t : 0;
      total += t;
    }
    kept += total;
    if (kept > cap) return false;                          // (the same for the whole workgroup)
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (take >> i & 1u) list[at++] = make_float2(x[i], __int_as_float(base + i));
    __syncthreads();
  }
  if (kept < ksel) return false;                           // (cannot be: tops and scores do not belong together)
  select_list<NT>(sm, list, kept, ksel, cut, thr_out, out);
  return true;
}

// The same for long rows.  One workgroup works on a head, so what counts is instructions per element: here about 30 (the
// select above: about 120).  The n scores of the head (thread t: elements u*NT + t, from memory) are laid on a histogram
// linear between the smallest and the largest (bins that follow the distance from a bound would pile the bulk of a full
// row into a few dozen of them); what lies in the bin of the ksel-th best or above, and what reaches a little below it,
// goes to LDS, ascending in position, as (score, element) pairs, and the select above finishes on those.  False if more
// than cap elements would go there: nothing has been written then.
template <int NT, int E, typename Out>
__device__ __forceinline__ bool select_long(SelectShared<NT>& sm, const float* __restrict__ sc, int n, int ksel,
                                            float2* list, int cap, float* __restrict__ thr_out, Out out) {
  constexpr int kWaves = NT / 64, kBins = 2 * NT;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  n = __builtin_amdgcn_readfirstlane(n);
  auto mine = [&](int u) { return tid < n - u * NT; };
  float v[E];                                              // (elements past the end: -inf, below every sanitised score)
#pragma unroll
  for (int u = 0; u < E; ++u) {
    const float* at = sc + u * NT;
    v[u] = mine(u) ? at[tid] : -INFINITY;
  }
  float hi = -FLT_MAX, mn = FLT_MAX;
#pragma unroll
  for (int u = 0; u < E; ++u) {
    const bool in = mine(u);
    v[u] = in ? sanitize(v[u]) : -INFINITY;
    hi = fmaxf(hi, v[u]);
    mn = in ? fminf(mn, v[u]) : mn;
  }
  hi = row16_max(hi);
  hi = fmaxf(hi, __shfl_xor(hi, 16));
  hi = fmaxf(hi, __shfl_xor(hi, 32));
  mn = -row16_max(-mn);
  mn = fminf(mn, __shfl_xor(mn, 16));
  mn = fminf(mn, __shfl_xor(mn, 32));
  if (lane == 0) {
    sm.whi[wv] = hi;
    sm.wlo[wv] = mn;
  }
  for (int i = tid; i < kBins; i += NT) sm.hist[i] = 0u;
  if (tid == 0) sm.list_n = 0u;
  __syncthreads();
  float lo = sm.wlo[0], top = sm.whi[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) {
    lo = fminf(lo, sm.wlo[w]);
    top = fmaxf(top, sm.whi[w]);
  }
  const float range = top - lo;
  const float scale = range > 0.f && range < FLT_MAX ? (float)kBins / range : 0.f;
#pragma unroll
  for (int u = 0; u < E; ++u)
    if (mine(u)) atomicAdd(&sm.hist[min((uint32_t)(int)((v[u] - lo) * scale), (uint32_t)(kBins - 1))], 1u);
  __syncthreads();
  find_bin(sm, (uint32_t)ksel, tid, lane, wv);
  // Every score x in the bin or above has (x - lo) * scale >= bin up to two roundings, 2.4e-4 bins: the real number
  // lo + (bin - 0.01) / scale is below x, and so is the nearest float, x being one.
  const float cut = scale > 0.f ? fmaxf(lo + ((float)sm.bin - 0.01f) / scale, -FLT_MAX) : -FLT_MAX;
  auto keep = [&](int u) { return v[u] >= cut; };
  int my_count = 0;                                        // lane u: what my wave keeps of its elements u
#pragma unroll
  for (int u = 0; u < E; ++u) {
    const int cnt = (int)__popcll(__ballot(keep(u)));
    my_count = lane == u ? cnt : my_count;
  }
  __syncthreads();                                         // everybody has read the histogram
  if (lane < E) sm.hist[lane * kWaves + wv] = (uint32_t)my_count;
  __syncthreads();
  constexpr int kRows = (E * kWaves + 63) / 64;
  int before[kRows];                                       // exclusive prefix of count 64 i + lane
  int carry = 0;
#pragma unroll
  for (int i = 0; i < kRows; ++i) {
    const int x = 64 * i + lane < E * kWaves ? (int)sm.hist[64 * i + lane] : 0;
    const int inc = wave_inclusive_sum(x);
    before[i] = carry + inc - x;
    carry += __builtin_amdgcn_readlane(inc, 63);
  }
  const int kept = carry;
  if (kept > cap) return false;                            // (the same for the whole workgroup)
#pragma unroll
  for (int u = 0; u < E; ++u) {
    const bool k = keep(u);
    const uint64_t m = __ballot(k);
    const int at = __builtin_amdgcn_readlane(before[u * kWaves / 64], (u * kWaves) % 64 + wv);
    if (k) list[at + lanes_below(m)] = make_float2(v[u], __int_as_float(u * NT + tid));
  }
  __syncthreads();
  select_list<NT>(sm, list, kept, ksel, cut, thr_out, out);
  return true;
}

}  // namespace lfps
