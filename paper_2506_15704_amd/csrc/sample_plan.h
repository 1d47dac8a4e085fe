// The sample of an exact Top-k (exact_topk.hip): arithmetic only, so that a test can compile it by itself.
#pragma once
#include <math.h>

#include "wide_cut.h"

namespace lfps {

// Rows of a group that are scored first, spread evenly, and the rank of the sample score that becomes the head's threshold.
struct SamplePlan {
  int ns, rank;
};
constexpr int kSampleRanks = 32;             // ranks that the sample's select has room for whatever the budget

// n: rows, k: the budget, both of a request; ranks: the largest rank there is room for, at least kSampleRanks and the budget.
// With p = k / n the rows of the whole context above the r-th best of ns sampled scores number about n r / ns, with a relative spread of
// 1 / sqrt(r).  That count must land between k (else too few survive) and the select's list capacity.  It is aimed at t k: 2 k or, of
// smaller budgets, 10 sqrt(n) and at most 2048 rows, but not past the middle of the two limits, t = (1 + cap / k) / 2; r is made large
// enough for both to lie z = 4.5 standard deviations away (a miss costs a rescoring of that head, never a wrong result), and the sample size
// follows as ns = (r / t) n / k.  A context no larger than that is sampled whole, with r = k; one of which more than ns_max rows were
// wanted has the rank that aims at t k.
// (A survivor costs a quarter of a sampled row or less.  Aimed at 2 k whatever the budget, small ones wanted more rows than the lists of
// candidates were wide, which the sample was kept to, and heads were left short in most calls.  With its attention, 8 requests with 8 x 4
// heads and 65536 rows, k = 8, 20, 72, 256, 500: 755, 772, 790, 209, 213 -> 198, 202, 201, 203, 207 us; 64 with 8 x 1 and 4608 rows, k = 20,
// 72, 256, radius 1: 206, 213, 146 -> 130, 134, 138.  Without the limit but aimed at 2 k: k = 72, radius 4 142 -> 178, aimed as now 135.)
LFPS_BOTH SamplePlan plan_sample(int n, int k, int ranks, int ns_max, int list_cap) {
  k = k < n ? k : n;
  int ns = n, r = k;
  if (k > 0 && n > k) {
    const float kf = (float)k, nf = (float)n;
    const float t = fminf(fmaxf(2.f, fminf(2048.f, 10.f * sqrtf(nf)) / kf), 0.5f * (1.f + (float)list_cap / kf));
    if (t > 1.05f) {                           // (else the list barely holds the budget: no room to aim)
      const int most = ns_max < n ? ns_max : n;
      const float sr = 4.5f * t / (t - 1.f);
      r = (int)ceilf(sr * sr);
      r = r < ranks ? r : ranks;
      const float want = ((float)r / t) * (nf / kf);
      if (want < (float)most) {
        ns = (int)ceilf(want);
      } else {
        ns = most;
        r = (int)(t * (float)ns * kf / nf);
      }
      if (ns >= n) {
        ns = n;
        r = k;
      }
    }
  }
  r = r < 1 ? 1 : r;
  r = r > ranks ? ranks : r;
  r = r > ns ? ns : r;
  return SamplePlan{ns, r};
}

}  // namespace lfps
