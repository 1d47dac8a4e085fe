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
    if (!strcmp(what, "plan")) {                    // requests, KV heads, rows, heads per group, pieces -> rows of a narrow range; the wide plan
      int batch, heads, rows, of_group, pieces;
      if (scanf("%d %d %d %d %d", &batch, &heads, &rows, &of_group, &pieces) != 5) return 1;
      const WidePlan p = wide_plan_for(batch, heads, rows, pieces);
      printf("%d %d %d %d %d\n", range_rows_for((long long)batch * heads, rows, of_group, false), p.rows, p.parts, p.slots, p.most);
    } else if (!strcmp(what, "share")) {            // slots, most, requests, then (rows, candidates) of each -> 0, or the parts of each
      int slots, most, batch, spare; float all = 0.f, largest = 0.f;
      if (scanf("%d %d %d", &slots, &most, &batch) != 3) return 1;
      std::vector<int> n(batch); std::vector<float> rows(batch);
      spare = slots;
      for (int i = 0; i < batch; ++i) {
        if (scanf("%d %f", &n[i], &rows[i]) != 2) return 1;
        all += rows[i];
        largest = largest > rows[i] ? largest : rows[i];
        spare -= fewest_parts(n[i]);
      }
      if (!uneven(largest, all, batch)) printf("0");
      else for (int i = 0; i < batch; ++i) printf("%d ", parts_of_request(n[i], rows[i], all, spare, most));
      printf("\n");
    } else if (!strcmp(what, "grid")) {             // requests, KV heads, rows, pieces -> its depth; slots and parts that are not one workgroup's
      int batch, heads, rows, pieces; long long bad = 0;
      if (scanf("%d %d %d %d", &batch, &heads, &rows, &pieces) != 4) return 1;
      const WidePlan p = wide_plan_for(batch, heads, rows, pieces);
      if (!p.rows) { printf("0 0\n"); continue; }
      const WideGrid grid = wide_grid(p, batch, heads);
      const int slots = p.slots > batch * p.parts ? p.slots : batch * p.parts;
      std::vector<int> even((size_t)batch * heads * p.parts), uneven((size_t)heads * slots);
      for (int z = 0; z < grid.deep; ++z) for (int y = 0; y < grid.parts; ++y) for (int x = 0; x < grid.beside; ++x) {
        const WideBlock block(batch * heads, heads, grid.beside, grid.parts, x, y, z);
        const int slot = block.slot(batch, heads, p.parts);
        if (!block.extra) ++even[((size_t)block.b * heads + block.g) * p.parts + block.part];
        if (slot < slots) ++uneven[(size_t)block.g * slots + slot];
      }
      for (int n : even) bad += n != 1;
      for (int n : uneven) bad += n != 1 && p.slots > 0;
      printf("%d %lld\n", grid.deep, bad);
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
          if (in.touches(i)) for (int y = in.from(i, r, in.begin); y <= in.to(i, r, in.begin, in.end); ++y) printf("%d ", s.row_of(x * s.rows + y));
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
        text = "\n".join(what + " " + " ".join(str(x) for x in c) for c in cases)
        res = subprocess.run([str(where / "cut")], input=text, capture_output=True, text=True, check=True)
        return [[int(x) for x in line.split()] for line in res.stdout.splitlines()]
    return ask


def _strip_rows(n, parts):
    return max(64, (-(-n // (2 * parts)) + 63) // 64 * 64)


def _pieces(L):
    """Piece counts that a head has room for whatever the form: of the exact Top-k's pass over all rows."""
    return L // ((-(-L // 1000) + 63) // 64 * 64) + 2


def test_plans_are_what_the_kernel_can_take(cut):
    rows = sorted({x + d for e in range(21) for x in (1 << e, 3 << e) for d in (-65, -1, 0, 1, 63) if 0 < x + d <= 88 * 1024 * 8})
    cases = [(B, h, n, 4, _pieces(n)) for B, h in [(g, 1) for g in list(range(1, 70)) + [127, 171, 256, 4096, 65535]] +
             [(1, 8), (2, 8), (16, 8), (21, 8), (32, 8), (33, 8), (48, 8), (49, 8), (64, 8), (65, 8), (1024, 8), (5, 3)] for n in rows]
    for (B, heads, n, _, pieces), (_, r, parts, slots, most) in zip(cases, cut("plan", cases)):
        groups = B * heads
        if r == 0:
            assert n > 65536 - 128 and groups > 8, (groups, n)
            continue
        assert r <= 65536 and r % 128 == 0 and 1 <= parts <= 128, (groups, n, r, parts)       # eight pieces each, 1024 per head
        assert parts <= most <= 128 and 8 * most <= max(pieces, 8 * parts)
        fewest = -(-n // 65536)
        assert fewest <= parts and (slots >= max(B * parts, B * fewest + 256 // heads) if B > 1 else slots == 0), (B, heads, n, slots)
        for m in {x for x in (1, 63, 64, 65, n // 3 + 1, n - 1, n) if 0 < x <= n}:     # a request's own strips: no longer ones
            assert 2 * _strip_rows(m, parts) <= r, (groups, n, m)
            assert 2 * _strip_rows(m, -(-m // 65536)) <= 65536


# (a grid may be 65535 deep; a batch has up to 65535 groups)
def test_grids_have_every_part_once(cut):
    cases = [(B, h, n, _pieces(n)) for B, h in [(g, 1) for g in (1, 2, 7, 8, 9, 63, 100, 257, 264, 385, 513, 700, 65528, 65529, 65535)] +
             [(1, 8), (1, 601), (1, 65535), (3, 5), (13, 5), (16, 8), (32, 8), (33, 8), (65, 8), (107, 5), (1024, 8), (4681, 14), (2, 32767), (9362, 7)]
             for n in (18, 33000, 65536, 140000)]
    for case, (deep, bad) in zip(cases, cut("grid", cases)):
        assert bad == 0 and deep <= 65535, (case, deep, bad)


def _candidates(n, k, r):
    """As the kernel estimates them, of four heads a group."""
    return n * (1 - np.exp(-1.6 * (2 * r + 2) * k / n))


# requests of uneven work, by length or by budget: none of the workgroups has more than its share many times over (cut evenly, the long
# request's would have 15 to 33), and there are as many as the launch has
@pytest.mark.parametrize("B,Hkv,L,lens,ks", [
    (32, 8, 100000, [100000] + [2000] * 31, [2000] + [40] * 31), (16, 8, 131072, [131072] + [4096] * 15, [2048] + [64] * 15),
    (128, 8, 32768, [1000] * 127 + [32768], [32] * 127 + [1024]), (32, 8, 65536, [65536] * 32, [64] * 9 + [4096] + [64] * 22),
    (8, 8, 65536, [1000] * 7 + [65536], [32] * 7 + [2048]),
    (64, 8, 32768, [max(1000, int(32768 * 0.9 ** i)) for i in range(64)], [max(16, int(655 * 0.9 ** i)) for i in range(64)])])
def test_uneven_requests_share_the_workgroups(cut, B, Hkv, L, lens, ks):
    ((narrow, r, parts, slots, most),) = cut("plan", [(B, Hkv, L, 4, _pieces(L))])
    assert narrow == 0 and r > 0
    rows = [_candidates(n, k, 4) for n, k in zip(lens, ks)]
    (got,) = cut("share", [[slots, most, B] + [x for nr in zip(lens, rows) for x in nr]])
    assert len(got) == B and sum(got) <= slots and min(got) >= 1
    load = max(x / p for x, p in zip(rows, got)) * 512 / Hkv / sum(rows)      # in shares of the chip's 512
    even = max(rows) / parts * 512 / Hkv / sum(rows)
    assert load < 0.5 * even and load < 4.5, (load, even)


def test_shares_are_never_more_than_there_are(cut):
    rng = np.random.default_rng(3)
    cases = []
    for _ in range(500):
        B, Hkv, L = int(rng.integers(2, 400)), int(rng.choice([1, 2, 4, 8])), int(64 * 11000 ** rng.random())
        cases.append((B, Hkv, L, [max(1, int(L * x)) for x in rng.random(B) ** rng.integers(1, 9)], rng.random(B) ** rng.integers(1, 20)))
    plans = cut("plan", [(B, Hkv, L, 4, _pieces(L)) for B, Hkv, L, _, _ in cases])
    took = [(c, p) for c, p in zip(cases, plans) if p[1]]
    shares = cut("share", [[p[3], p[4], c[0]] + [x for nr in zip(c[3], (n * f for n, f in zip(c[3], c[4]))) for x in nr] for c, p in took])
    assert len(took) > 100 and sum(len(x) > 1 for x in shares) > 50
    for (c, p), got in zip(took, shares):
        if len(got) > 1:
            assert sum(got) <= p[3] and max(got) <= p[4]
            assert all(2 * _strip_rows(n, parts) <= 65536 for n, parts in zip(c[3], got))


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
    ((narrow, r, parts, _, _),) = cut("plan", [(B, Hkv, L, 4, _pieces(L))])
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
    got = cut("plan", [(B, Hkv, L + 6, Hq // Hkv, _pieces(L + 6)) for B, Hq, Hkv, L, *_ in STEPS])
    assert all(narrow == 0 and r > 0 for narrow, r, *_ in got)
    assert {x[2] for x in got} >= {1, 2, 4, 32, 64, 128} and max(x[1] for x in got) == 65024
    # of the last one the candidates outgrow 256 MiB: heads' windows of 2 r + 2 rows around k random rows, 256 bytes each
    B, Hq, Hkv, L, k, r = STEPS[-1][:6]
    assert B * Hkv * L * (1 - np.exp(-(2 * r + 2) * k / L)) * 256 > 256 << 20


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,L,k,r,n_recent,n_sink,dtype,page", STEPS)
def test_steps(B, Hq, Hkv, L, k, r, n_recent, n_sink, dtype, page):
    from tests.test_gpu_ranges import test_memoryless_steps as steps
    steps(B, Hq, Hkv, L, k, r, n_recent, n_sink, dtype, page)


# many groups, no multiple of eight: of one request, and of many
@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,L,k,r,n_recent,n_sink,dtype,page", [(1, 601, 601, 2100, 40, 2, 0, 4, "bf16", 0),
                                                                       (171, 6, 3, 2100, 40, 2, 0, 4, "fp8", 16)])
def test_many_groups(B, Hq, Hkv, L, k, r, n_recent, n_sink, dtype, page, cut):
    ((narrow, rows, parts, *_),) = cut("plan", [(B, Hkv, L, Hq // Hkv, _pieces(L))])
    assert narrow == 0 and rows > 0 and parts == 1
    test_steps(B, Hq, Hkv, L, k, r, n_recent, n_sink, dtype, page)


# one long request among short ones and of one row, one large budget among small ones, a request that needs two workgroups for its places,
# more requests than a wave has lanes, many groups, no multiple of eight: against an unfiltered context, and the same bits when the batch changes between steps
@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,L,lens,ks,dtype,page", [
    (3, 3, 6000, [100] * 150 + [6000] + [33] * 20, [9] * 150 + [400] + [3] * 20, "bf16", 0),
    (8, 8, 100000, [100000, 1, 2000, 64, 65] + [700] * 7, [1500, 1, 40, 5, 64] + [30] * 7, "bf16", 0),
    (32, 8, 140000, [300, 139000, 20000], [20, 1000, 300], "fp8", 16), (16, 8, 16500, [16500] * 9, [30] * 8 + [900], "f16", 64),
    (4, 4, 6000, [100] * 69 + [6000] + [33] * 7, [9] * 69 + [400] + [3] * 7, "bf16", 16)])
def test_uneven_steps(Hq, Hkv, L, lens, ks, dtype, page, cut):
    import torch
    from tests.harness import DEV
    from tests.test_gpu_ranges import _cache, _pair, _view
    B, k = len(lens), max(ks)
    ((narrow, r, parts, slots, most),) = cut("plan", [(B, Hkv, L, Hq // Hkv, _pieces(L))])
    assert narrow == 0 and r > 0
    heads = {1: 1.0, 2: 1.3, 4: 1.6}[Hq // Hkv]
    rows = [n - (n - 1) * np.exp(-heads * 10 * x / n) for n, x in zip(lens, ks)]
    assert len(cut("share", [[slots, most, B] + [x for nr in zip(lens, rows) for x in nr]])[0]) == B          # (uneven)
    g = torch.Generator(device=DEV)
    g.manual_seed(L + k)
    cache = _cache(B, Hkv, L, dtype, page, g)
    a, b = _pair(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="bf16" if dtype == "fp8" else dtype, k_fp8=dtype == "fp8", max_seq_len=L,
                 max_k=k, radius=4)
    q = torch.randn((B, Hq, 128), device=DEV, generator=g)
    prev = torch.full((B, Hq, k), -1, dtype=torch.int32, device=DEV)
    kt = torch.tensor(ks, dtype=torch.int32, device=DEV)
    a.lfps_exact_topk(q, _view(a, cache, torch.tensor(lens, dtype=torch.int32, device=DEV)), kt, prev)
    for t in range(4):
        q = q * 0.02 if t == 3 else q + 0.1 * torch.randn((B, Hq, 128), device=DEV, generator=g)
        seq = torch.tensor(lens if t != 2 else [min(lens)] * B, dtype=torch.int32, device=DEV)        # (an even batch in between)
        res = []
        for ctx in (a, b):
            idx = torch.full((B, Hq, k), -5, dtype=torch.int32, device=DEV)
            sc, out = torch.full((B, Hq, k), -5.0, device=DEV), torch.full((B, Hq, 128), -5.0, device=DEV)
            cnt = torch.full((B, Hkv), -5, dtype=torch.int32, device=DEV)
            ctx.lfps_step(q, _view(ctx, cache, seq), prev, kt, idx, out, sc)
            ctx.lfps_copy_cand_count(cnt)
            assert ctx.lfps_poll_status() == 0
            res.append((idx, sc, out, cnt))
        for x, y, name in zip(*res, ("index", "score", "output", "candidate count")):
            assert torch.equal(x, y), (name, t, int((x != y).sum()))
        if t != 2:
            prev = res[0][0]
    a.close()
    b.close()


# a NaN query and infinite ones: rows of the request, distinct and as many as the budget, for their groups; what a clean step gives for the others
@pytest.mark.gpu
@pytest.mark.parametrize("Hkv,L,dtype", [(8, 66000, "bf16"), (8, 66000, "f16"), (4, 140000, "fp8")])
def test_non_finite_queries(Hkv, L, dtype, cut):
    import torch
    from tests.harness import DEV
    from tests.test_gpu_ranges import _cache, _pair, _view
    B, Hq, k = 2, 4 * Hkv, 300
    ((narrow, r, *_),) = cut("plan", [(B, Hkv, L, 4, _pieces(L))])
    assert narrow == 0 and r > 0
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    cache = _cache(B, Hkv, L, dtype, 0, g)
    clean, dirty = _pair(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="bf16" if dtype == "fp8" else dtype, k_fp8=dtype == "fp8",
                         max_seq_len=L, max_k=k, radius=3)
    dirty.lfps_set_filter(True)
    seq, ks = (torch.tensor([x] * B, dtype=torch.int32, device=DEV) for x in (L, k))
    q = torch.randn((B, Hq, 128), device=DEV, generator=g)
    prev = torch.full((B, Hq, k), -1, dtype=torch.int32, device=DEV)
    clean.lfps_exact_topk(q, _view(clean, cache, seq), ks, prev)
    before = [prev, prev]
    for t in range(3):
        q = q + 0.1 * torch.randn((B, Hq, 128), device=DEV, generator=g)
        bad = q.clone()
        bad[0, 1, 5], bad[0, Hq - 1, :], bad[1, 6, 100] = float("nan"), float("inf"), float("-inf")
        res = []
        for ctx, query, last in ((clean, q, before[0]), (dirty, bad, before[1])):
            idx, out = torch.full((B, Hq, k), -5, dtype=torch.int32, device=DEV), torch.zeros((B, Hq, 128), device=DEV)
            ctx.lfps_step(query, _view(ctx, cache, seq), last, ks, idx, out)
            res.append((idx, out))
        before = [res[0][0], res[1][0]]
        groups = {(0, 0), (0, Hkv - 1), (1, 1)}
        for b in range(B):
            for h in range(Hq):
                mine = res[1][0][b, h]
                if (b, h // 4) in groups:
                    assert int(mine.min()) >= 0 and int(mine.max()) < L and len(torch.unique(mine)) == k, (t, b, h)
                else:
                    assert torch.equal(mine, res[0][0][b, h]) and torch.equal(res[1][1][b, h], res[0][1][b, h]), (t, b, h)
    clean.close()
    dirty.close()


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
