"""The register select of the chained steps at the edges of its dispatch (threads per head, elements per thread, ties,
crowded bins, lists that do not fit): bit for bit against the stand-alone select and attention on the same candidates,
which other tests hold against the oracle."""
import numpy as np
import pytest
import torch

from tests.harness import DEV

pytestmark = pytest.mark.gpu


def _reference(ctx, q, kv, prev, k, seq):
    """The same step through the separate entry points."""
    B, Hq, Hkv = ctx.B, ctx.Hq, ctx.Hkv
    cand = torch.zeros((B, Hkv, ctx.cand_cap), dtype=torch.int32, device=DEV)
    cnt = torch.zeros((B, Hkv), dtype=torch.int32, device=DEV)
    idx = torch.full((B, Hq, ctx.kmax), -7, dtype=torch.int32, device=DEV)
    sc = torch.full((B, Hq, ctx.kmax), -7.0, device=DEV)
    out = torch.full((B, Hq, 128), -7.0, device=DEV)
    ctx.lfps_candidates(prev, k, seq, cand, cnt)
    ctx.lfps_score_topk(q, kv, cand, cnt, k, idx, sc)
    ctx.lfps_sparse_attn(q, kv, idx, sc, k, out)
    return idx, sc, out


# heads: up to 256 -> 1024 threads, up to 512 -> 512, more -> 256 (unless the budget needs more); budgets that put the
# survivors on both sides of 2, 4, 8 and 16 elements per thread; dtype f32 = the select from full score rows
@pytest.mark.parametrize("B,Hq,Hkv,L,k,r,dtype", [
    (1, 4, 1, 3000, 63, 2, "bf16"), (1, 4, 1, 3001, 1, 0, "bf16"), (2, 8, 2, 6000, 1600, 3, "bf16"),
    (2, 8, 4, 9000, 3300, 3, "f16"), (1, 8, 2, 30000, 9000, 1, "bf16"), (8, 64, 16, 1500, 400, 3, "bf16"),
    (8, 64, 16, 5000, 900, 3, "bf16"), (8, 64, 16, 5000, 1700, 2, "bf16"), (17, 32, 8, 900, 200, 3, "bf16"),
    (17, 32, 8, 2500, 450, 3, "f16"), (17, 32, 8, 3500, 1500, 2, "bf16"), (17, 32, 8, 5000, 2100, 1, "bf16"),
    (2, 8, 2, 900, 100, 2, "f32"), (2, 8, 2, 9000, 700, 4, "f32"), (1, 8, 2, 24000, 4000, 4, "f32"),
    (1, 8, 2, 40000, 12000, 2, "f32")])
@pytest.mark.parametrize("values", ["normal", "ties"])
def test_step_equals_the_separate_calls(B, Hq, Hkv, L, k, r, dtype, values):
    from paper_2506_15704_amd.binding import Lfps
    g = torch.Generator(device=DEV)
    g.manual_seed(B * 1000 + L)
    dt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[dtype]
    Lcap = L + 8
    K = torch.randn((B, Hkv, Lcap, 128), device=DEV, generator=g)
    if values == "ties":           # rows from a small set: long runs of equal scores at every cut
        K = K[:, :, : max(3, L // 700)][:, :, torch.randint(0, max(3, L // 700), (Lcap,), device=DEV, generator=g)].contiguous()
    K = K.to(dt)
    V = torch.randn((B, Hkv, Lcap, 128), device=DEV, generator=g).to(dt)
    ctx = Lfps(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype=dtype, max_seq_len=Lcap, max_k=k, radius=r)
    lens = [max(1, L - 37 * b) for b in range(B)]
    ks = torch.tensor([max(1, min(k - 5 * b, n)) if b else k for b, n in enumerate(lens)], dtype=torch.int32, device=DEV)
    q = torch.randn((B, Hq, 128), device=DEV, generator=g)
    prev = torch.full((B, Hq, k), -1, dtype=torch.int32, device=DEV)
    seq = torch.tensor(lens, dtype=torch.int32, device=DEV)
    ctx.lfps_exact_topk(q, ctx.kv_view(K, V, seq), ks, prev)
    for t in range(1, 4):          # the first step takes the unfiltered kernels, the later ones the filtered
        q = q + 0.05 * torch.randn((B, Hq, 128), device=DEV, generator=g)
        seq = torch.tensor([n + t for n in lens], dtype=torch.int32, device=DEV)
        kv = ctx.kv_view(K, V, seq)
        idx = torch.full((B, Hq, k), -5, dtype=torch.int32, device=DEV)
        sc = torch.full((B, Hq, k), -5.0, device=DEV)
        out = torch.full((B, Hq, 128), -5.0, device=DEV)
        want = _reference(ctx, q, kv, prev, ks, seq)
        ctx.lfps_step(q, kv, prev, ks, idx, out, sc)
        for got, ref, name in zip((idx, sc, out), want, ("index", "score", "output")):
            assert torch.equal(got, ref), (name, t, int((got != ref).sum()))
        prev = idx
    ctx.close()


# the stand-alone select: 4, 8, 16 and 32 scores per thread of its 1024, one more, and the streamed form
@pytest.mark.parametrize("L,k", [(1, 1), (63, 63), (4096, 100), (4097, 4097), (8191, 1), (8193, 700), (16384, 16384),
                                 (16385, 2000), (32767, 1024), (32768, 1023), (32769, 5000)])
@pytest.mark.parametrize("values", ["spread", "few", "equal", "outlier"])
def test_stand_alone_select(L, k, values):
    """Keys and queries of small whole numbers: dot products are exact, so the selection is fixed (equal scores at the
    cut go to the lower position)."""
    from paper_2506_15704_amd.binding import Lfps
    g = torch.Generator(device=DEV)
    g.manual_seed(L + k)
    ints = lambda lo, hi, shape: torch.randint(lo, hi, shape, device=DEV, generator=g).float()
    Hq, Hkv = 4, 1
    K = ints(-3, 4, (1, Hkv, L, 128)) if values == "spread" else ints(-1, 2, (1, Hkv, L, 128))
    q = ints(-8, 9, (1, Hq, 128))
    if values == "few":
        K[..., 2:] = 0
    if values == "equal":
        K[:] = 1
    if values == "outlier":
        K[0, 0, L // 2] = 100 * q[0, 0]
    ctx = Lfps(batch=1, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="f32", max_seq_len=L, max_k=k, radius=1)
    seq, kk = (torch.tensor([x], dtype=torch.int32, device=DEV) for x in (L, k))
    idx = torch.full((1, Hq, k), -5, dtype=torch.int32, device=DEV)
    sc = torch.full((1, Hq, k), -5.0, device=DEV)
    ctx.lfps_exact_topk(q, ctx.kv_view(K, K, seq), kk, idx, sc)
    dots = (q[0].double() @ K[0, 0].double().T).cpu()
    order = torch.sort(dots, dim=1, descending=True, stable=True).indices[:, :k].sort(dim=1).values
    assert torch.equal(idx[0].cpu().long(), order)
    want = (torch.gather(dots, 1, order).float() * torch.tensor(0.08838834764831845, dtype=torch.float32))
    assert torch.equal(sc[0].cpu(), want)
    ctx.close()


def test_many_heads_hold_survivors_of_several_budgets():
    """544 heads, each with more than two budgets of survivors (larger queries than the step before): they fit the select's
    list, and no head is scored again."""
    from paper_2506_15704_amd.binding import Lfps
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    B, Hq, Hkv, L, k = 17, 32, 8, 12000, 2048
    K = torch.randn((B, Hkv, L + 8, 128), device=DEV, generator=g).to(torch.bfloat16)
    ctxs = [Lfps(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="bf16", max_seq_len=L + 8, max_k=k, radius=4) for _ in range(2)]
    ctxs[1].lfps_set_filter(False)
    ks = torch.full((B,), k, dtype=torch.int32, device=DEV)
    q = torch.randn((B, Hq, 128), device=DEV, generator=g)
    prev = torch.zeros((B, Hq, k), dtype=torch.int32, device=DEV)
    ctxs[0].lfps_exact_topk(q, ctxs[0].kv_view(K, K, torch.full((B,), L, dtype=torch.int32, device=DEV)), ks, prev)
    ctxs[0].lfps_poll_rescored()
    for t, scale in ((1, 1.0), (2, 3.0)):
        seq = torch.full((B,), L + t, dtype=torch.int32, device=DEV)
        res = []
        for ctx in ctxs:
            idx, out = torch.zeros((B, Hq, k), dtype=torch.int32, device=DEV), torch.zeros((B, Hq, 128), device=DEV)
            ctx.lfps_step(scale * q, ctx.kv_view(K, K, seq), prev, ks, idx, out)
            res.append((idx, out))
        assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1]), t
        assert ctxs[0].lfps_poll_rescored() == 0, t
    for ctx in ctxs:
        ctx.close()
