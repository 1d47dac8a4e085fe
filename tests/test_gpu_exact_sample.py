"""The sample from which the exact Top-k of large contexts takes its thresholds, and what is settled beside its scores: the same Top-k as
from all scores, for samples that are all rows, a part of them, and of requests of one row, with more requests than a wave has lanes."""
import pytest
import torch

from tests.harness import DEV
from tests.test_gpu_ranges import _cache, _pair, _view

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,L,k,dtype,page", [
    (66, 8, 8, 2000, 30, "bf16", 0), (5, 32, 8, 30000, 400, "f16", 16), (2, 4, 2, 270000, 700, "fp8", 0), (17, 16, 8, 8000, 3000, "bf16", 64)])
def test_exact_topk(B, Hq, Hkv, L, k, dtype, page):
    g = torch.Generator(device=DEV)
    g.manual_seed(L + k)
    cache = _cache(B, Hkv, L, dtype, page, g)
    lens = [max(1, L - (L // 7 + 1) * (i % 9)) for i in range(B)]
    seq = torch.tensor(lens, dtype=torch.int32, device=DEV)
    ks = torch.tensor([max(1, min(k - i % 5, n)) for i, n in enumerate(lens)], dtype=torch.int32, device=DEV)
    q = torch.randn((B, Hq, 128), device=DEV, generator=g)
    res = []
    for ctx in _pair(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="bf16" if dtype == "fp8" else dtype, k_fp8=dtype == "fp8",
                     max_seq_len=L, max_k=k, radius=1):
        idx, sc = torch.full((B, Hq, k), -5, dtype=torch.int32, device=DEV), torch.full((B, Hq, k), -5.0, device=DEV)
        ctx.lfps_exact_topk(q, _view(ctx, cache, seq), ks, idx, sc)
        assert ctx.lfps_poll_status() == 0
        res.append((idx, sc))
        ctx.close()
    for x, y in zip(*res):
        assert torch.equal(x, y)
