"""Wide ranges: candidates and scores in one kernel for chained steps of more than a million rows, where a request's rows are cut into
equal parts.  The rule by itself, and the steps against an unfiltered context, which takes other kernels."""
import shutil
import subprocess

import pytest

from paper_2506_15704_amd import build

MAIN = r"""
#include <cstdio>
#include "range_rule.h"
int main() {
  long long groups; int rows;
  while (scanf("%lld %d", &groups, &rows) == 2) printf("%d\n", lfps::wide_rows_for(groups, rows));
}
"""


def test_wide_ranges_are_what_the_kernel_can_take(tmp_path):
    (tmp_path / "main.cpp").write_text(MAIN)
    compiler = shutil.which("g++") or build.hipcc()
    subprocess.run([compiler, "-std=c++17", "-O1", "-I", build.CSRC, str(tmp_path / "main.cpp"), "-o", str(tmp_path / "rule")], check=True)
    rows = sorted({x + d for e in range(21) for x in (1 << e, 3 << e) for d in (-65, -1, 0, 1, 63) if 0 < x + d <= 88 * 1024 * 8})
    cases = [(g, n) for g in list(range(1, 70)) + [127, 128, 170, 171, 256, 257, 384, 385, 512, 513, 1024, 4096, 65535] for n in rows]
    res = subprocess.run([str(tmp_path / "rule")], input="\n".join("%d %d" % c for c in cases), capture_output=True, text=True, check=True)
    for (groups, n), r in zip(cases, [int(x) for x in res.stdout.split()]):
        if r == 0:
            assert n > 65536 and groups > 8, (groups, n)
            continue
        assert r % 64 == 0 and 64 <= r <= 65536, (groups, n, r)
        parts = -(-n // r)
        assert parts <= 256, (groups, n, r)                      # four pieces each, 1024 per head
        for m in {x for x in (1, 63, 64, 65, n // 3 + 1, n - 1, n) if 0 < x <= n}:     # a request's own ranges: no more of them, and none longer
            own = max(64, (-(-m // parts) + 63) // 64 * 64)
            assert own <= r and -(-m // own) <= parts, (groups, n, m)


# one group whose ranges are limited by the pieces of a head; ranges of more than a word per thread; requests of one row beside full
# ones; two ranges per group beyond 256 groups and one beyond 512; radius 0 and one wider than a word of windows; rows past the caches
@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,L,k,r,n_recent,n_sink,dtype,page", [
    (1, 4, 1, 720000, 700, 3, 1, 0, "bf16", 0), (2, 2, 2, 300000, 2500, 0, 70, 5, "bf16", 0), (16, 16, 8, 33000, 129, 2, 1, 0, "f16", 64),
    (33, 32, 8, 4060, 60, 4, 1, 0, "bf16", 16), (65, 8, 8, 2100, 40, 2, 0, 4, "fp8", 16), (4, 32, 8, 40000, 900, 20, 1, 0, "fp8", 0),
    (1, 32, 8, 140000, 3000, 14, 1, 0, "bf16", 0)])
def test_steps(B, Hq, Hkv, L, k, r, n_recent, n_sink, dtype, page):
    from tests.test_gpu_ranges import test_memoryless_steps as steps
    steps(B, Hq, Hkv, L, k, r, n_recent, n_sink, dtype, page)


# requests that are far below the context's capacity have ranges of their own length: the same bits as in a context without that room
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
