"""The sample from which an exact Top-k takes its thresholds, compiled by itself: few heads are left short of rows, or with more than the
list holds."""
import math
import shutil
import subprocess

import pytest

from paper_2506_15704_amd import build

MAIN = r"""
#include <cstdio>
#include "sample_plan.h"
int main() {
  int n, k, kmax, cap;
  while (scanf("%d %d %d %d", &n, &k, &kmax, &cap) == 4) {
    const lfps::SamplePlan p = lfps::plan_sample(n, k, kmax, 32768, cap);
    printf("%d %d\n", p.ns, p.rank);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    where = tmp_path_factory.mktemp("plan")
    (where / "main.cpp").write_text(MAIN)
    compiler = shutil.which("g++") or build.hipcc()
    subprocess.run([compiler, "-std=c++17", "-O1", "-I", build.CSRC, str(where / "main.cpp"), "-o", str(where / "plan")], check=True)

    def ask(cases):
        res = subprocess.run([str(where / "plan")], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True, text=True,
                             check=True)
        return [tuple(int(x) for x in line.split()) for line in res.stdout.splitlines()]
    return ask


# (limited by the width of candidate lists and by the rank that a row of the budget holds, these were 289 and 9, 4608 and 20, ...)
def test_a_sample_is_as_large_as_its_rank_needs(plan):
    assert plan([(4608, 72, 128, 16384), (4608, 20, 32, 16384), (32768, 1024, 1024, 16384), (65536, 1024, 1024, 16384),
                 (65536, 72, 128, 16384), (65536, 1, 32, 16384)]) == [(177, 26), (150, 22), (1296, 81), (2592, 81), (704, 22), (672, 21)]


def test_samples_leave_few_heads_short(plan):
    cases = [(n, k, max(32, kmax), cap) for n in (1, 50, 700, 4608, 16384, 32768, 40000, 131072, 700000)
             for k in (1, 3, 15, 16, 20, 40, 41, 60, 72, 81, 130, 500, 513, 1023, 1024, 2048, 9000)
             for kmax in (k, 2 * k, 9000) for cap in (4096, 8192, 16384) if k <= kmax <= n and 1.25 * kmax <= cap]
    for (n, k, ranks, cap), (ns, rank) in zip(cases, plan(cases)):
        assert 1 <= rank <= min(ranks, ns) and 1 <= ns <= n
        if ns == n:
            assert rank == min(k, n)
            continue
        reach = n * rank / ns                                    # rows that reach the threshold, with a relative spread of 1 / sqrt(rank)
        spread = reach / math.sqrt(rank)
        if 100 < ns < 32768:                                       # (more were wanted, or few of few rows: whole rows are coarse then)
            assert (reach - k) / spread >= 4.3, (n, k, ranks, cap, ns, rank)
            assert (cap - reach) / spread >= 4.3, (n, k, ranks, cap, ns, rank)
