"""Candidates and scores in one kernel for chained steps of more than a million rows, where every workgroup has strips spread over its
request.  The cut by itself, and the steps against an unfiltered context, which takes other kernels."""
import shutil
import subprocess

import numpy as np
import pytest

from paper_2506_15704_amd import build

MAIN = r"""
#include <cstdio>
#include <cstring>
#include <vector>
#include "range_rule.h"
#include "wide_cut.h"
using namespace lfps;
int main() {
  char what[16];
  while (scanf("%15s", what) == 1) {
    if (!strcmp(what, "plan")) {                    // groups, rows, heads per group -> rows of a narrow range; the wide plan
      long long groups; int rows, heads;
      if (scanf("%lld %d %d", &groups, &rows, &heads) != 3) return 1;
      const WidePlan p = wide_plan_for(groups, rows);
      printf("%d %d %d\n", range_rows_for(groups, rows, heads, false), p.rows, p.parts);
    } else if (!strcmp(what, "rows")) {             // rows, parts: which rows are not one workgroup's, or not found again
      int n, parts; long long bad = 0;
      if (scanf("%d %d", &n, &parts) != 2) return 1;
      std::vector<int> owners(n);
      for (int part = 0; part < parts; ++part) {
        const Strips s(n, parts, part);
        for (int place = 0; place < 2 * s.rows; ++place) {
          const int row = s.row_of(place);
          if (row < n) ++owners[row];
          bad += row != (place < s.rows ? part * s.rows + place : (parts + part) * s.rows + place - s.rows);
        }
      }
      for (int x : owners) bad += x != 1;
      printf("%lld\n", bad);
    } else {                                        // window: rows, parts, entry, radius -> the rows that the parts mark
      int n, parts, i, r;
      if (scanf("%d %d %d %d", &n, &parts, &i, &r) != 4) return 1;
      for (int part = 0; part < parts; ++part) {
        const Strips s(n, parts, part);
        for (int x = 0; x < 2; ++x) {
          const StripWindows in(n, x ? s.second : s.first, s.rows, r);
          if (in.touches(i)) for (int y = in.from(i, r); y <= in.to(i, r); ++y) printf("%d ", s.row_of(x * s.rows + y));
        }
      }
      printf("\n");
    }
  }
}
"""


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    where = tmp_path_factory.mktemp("cut")
    (where / "main.cpp").write_text(MAIN)
    compiler = shutil.which("g++") or build.hipcc()
    subprocess.run([compiler, "-std=c++17", "-O1", "-I", build.CSRC, str(where / "main.cpp"), "-o", str(where / "cut")], check=True)

    def ask(what, cases):
        text = "\n".join(what + " " + " ".join(str(int(x)) for x in c) for c in cases)
        res = subprocess.run([str(where / "cut")], input=text, capture_output=True, text=True, check=True)
        return [[int(x) for x in line.split()] for line in res.stdout.splitlines()]
    return ask


def _strip_rows(n, parts):
    return max(64, (-(-n // (2 * parts)) + 63) // 64 * 64)


def test_plans_are_what_the_kernel_can_take(cut):
    rows = sorted({x + d for e in range(21) for x in (1 << e, 3 << e) for d in (-65, -1, 0, 1, 63) if 0 < x + d <= 88 * 1024 * 8})
    cases = [(g, n, 4) for g in list(range(1, 70)) + [127, 128, 170, 171, 256, 257, 384, 385, 512, 513, 1024, 4096, 65535] for n in rows]
    for (groups, n, _), (_, r, parts) in zip(cases, cut("plan", cases)):
        if r == 0:
            assert n > 65536 - 128 and groups > 8, (groups, n)
            continue
        assert r <= 65536 and r % 128 == 0 and 1 <= parts <= 128, (groups, n, r, parts)       # eight pieces each, 1024 per head
        for m in {x for x in (1, 63, 64, 65, n // 3 + 1, n - 1, n) if 0 < x <= n}:     # a request's own strips: no longer ones
            assert 2 * _strip_rows(m, parts) <= r, (groups, n, m)


@pytest.mark.parametrize("n,parts", [(1, 64), (70, 4), (4096, 1), (33006, 4), (140006, 64), (65024, 1), (131076, 4), (720896, 128), (5000, 3),
                                     (263000, 5), (129, 1)])
def test_every_row_is_one_workgroups(cut, n, parts):
    assert cut("rows", [(n, parts)]) == [[0]]
    rng = np.random.default_rng(n)
    at = [int(x) for x in rng.integers(0, n, 60)] + [0, n - 1]
    cases = [(n, parts, a, r) for a in at for r in (0, 2, 15, 90, 3000)]
    for (_, _, i, r), got in zip(cases, cut("window", cases)):
        assert sorted(got) == list(range(max(0, i - r), min(n - 1, i + r + 1) + 1)), (i, r)
    none = [(n, parts, i, r) for i in (-1, n, n + 1, 2**31 - 1, -2**31) for r in (0, 15, 3000, 1 << 20)]
    assert cut("window", none) == [[]] * len(none)


# Top-k rows that crowd in the last `part` of a request: with one piece of the rows for each workgroup one in `parts` has the work of all.
# Of the 512 workgroups at least 128 have some, on CUs of their own half of the chip, which takes rows in as fast as memory gives them.
@pytest.mark.parametrize("B,Hkv,L,part", [(8, 8, 32768, 0.125), (16, 8, 131072, 0.125), (16, 8, 131072, 0.25), (2, 8, 131072, 0.125),
                                          (32, 8, 65536, 0.125), (1, 8, 140000, 0.25)])
def test_crowded_rows_are_shared(cut, B, Hkv, L, part):
    ((narrow, r, parts),) = cut("plan", [(B * Hkv, L, 4)])
    assert narrow == 0 and r > 0
    crowd = np.arange(int(L * (1 - part)), L)
    load = np.bincount(crowd // _strip_rows(L, parts) % parts, minlength=parts)
    assert B * Hkv * (load > 0).sum() >= 128, load


# 64 workgroups per group, of one head; 128, all that a head has pieces for; requests of few rows beside full ones; two workgroups per group beyond 256 groups and one beyond 512, with places up to the last of 16 bits; radius 0 and one wider
# than a word of windows; rows past the caches
STEPS = [
    (1, 8, 8, 140000, 2000, 3, 1, 0, "bf16", 0), (2, 2, 2, 300000, 2500, 0, 70, 5, "bf16", 0), (2, 16, 8, 66000, 900, 3, 70, 5, "bf16", 0), (16, 16, 8, 33000, 129, 2, 1, 0, "f16", 64),
    (33, 32, 8, 4060, 60, 4, 1, 0, "bf16", 16), (65, 8, 8, 2100, 40, 2, 0, 4, "fp8", 16), (4, 32, 8, 40000, 900, 20, 1, 0, "fp8", 0),
    (1, 32, 8, 140000, 3000, 14, 1, 0, "bf16", 0), (65, 8, 8, 65000, 300, 4, 1, 0, "fp8", 0), (16, 8, 8, 33000, 1500, 4, 1, 0, "bf16", 0)]


def test_the_steps_below_are_wide(cut):
    got = cut("plan", [(B * Hkv, L + 6, Hq // Hkv) for B, Hq, Hkv, L, *_ in STEPS])
    assert all(narrow == 0 and r > 0 for narrow, r, _ in got)
    assert {p for _, _, p in got} >= {1, 2, 4, 32, 64, 128} and max(r for _, r, _ in got) == 65024
    # of the last one the candidates outgrow 256 MiB: heads' windows of 2 r + 2 rows around k random rows, 256 bytes each
    B, Hq, Hkv, L, k, r = STEPS[-1][:6]
    assert B * Hkv * L * (1 - np.exp(-(2 * r + 2) * k / L)) * 256 > 256 << 20


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,L,k,r,n_recent,n_sink,dtype,page", STEPS)
def test_steps(B, Hq, Hkv, L, k, r, n_recent, n_sink, dtype, page):
    from tests.test_gpu_ranges import test_memoryless_steps as steps
    steps(B, Hq, Hkv, L, k, r, n_recent, n_sink, dtype, page)


# requests that are far below the context's capacity have strips of their own length: the same bits as in a context without that room
@pytest.mark.gpu
def test_room_to_grow():
    import torch
    from paper_2506_15704_amd.binding import Lfps
    from tests.harness import DEV
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    n, k = 70, 20
    K, V = (torch.randn((1, 8, 140000, 128), device=DEV, generator=g).to(torch.bfloat16) for _ in range(2))
    q = torch.randn((1, 32, 128), device=DEV, generator=g)
    seq, ks = (torch.tensor([x], dtype=torch.int32, device=DEV) for x in (n, k))
    res = []
    for room in (n, 140000):
        ctx = Lfps(batch=1, max_seq_len=room, max_k=k, radius=2)
        kv = ctx.kv_view(K[:, :, :room], V[:, :, :room], seq)
        a, b, c = (torch.full((1, 32, k), -1, dtype=torch.int32, device=DEV) for _ in range(3))
        out = torch.zeros((1, 32, 128), device=DEV)
        ctx.lfps_exact_topk(q, kv, ks, a)
        ctx.lfps_step(q, kv, a, ks, b, out)
        ctx.lfps_step(q * 1.01, kv, b, ks, c, out)
        res.append((b, c, out))
        ctx.close()
    for x, y in zip(*res):
        assert torch.equal(x, y)
