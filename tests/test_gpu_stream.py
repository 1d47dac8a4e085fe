"""Passes over more rows than the memory-side cache holds, whose rows are fetched past the caches.  Scoring (rows turned into
operands in LDS): bit for bit what the unfiltered kernels return, which other tests hold against the oracle.  Full attention and
score tables: against the same rows when the call holds few."""
import pytest
import torch

from tests.harness import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,page,B,L,Hq,Hkv", [
    ("bf16", 0, 5, 40007, 32, 8), ("bf16", 16, 3, 70001, 16, 8), ("f16", 64, 5, 40013, 32, 8), ("f16", 0, 7, 33331, 8, 8),
    ("fp8k", 0, 5, 70003, 16, 8), ("fp8kv", 16, 6, 60011, 32, 8)])
def test_streamed_scoring_equals_the_unfiltered_kernels(dtype, page, B, L, Hq, Hkv):
    from paper_2506_15704_amd.binding import Lfps
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    kd = {"bf16": torch.bfloat16, "f16": torch.float16}.get(dtype, torch.float8_e4m3fn)
    vd = torch.bfloat16 if dtype == "fp8k" else kd
    Lcap, k, r = L + 4, L // 20, 12
    nb = -(-Lcap // page) if page else 1
    shape = (B * nb, Hkv, page, 128) if page else (B, Hkv, Lcap, 128)
    K, V = (torch.empty(shape, dtype=d, device=DEV) for d in (kd, vd))
    for T in (K, V):
        for i in range(0, shape[0], -(-shape[0] // B)):
            T[i:i + -(-shape[0] // B)] = torch.randn(T[i:i + -(-shape[0] // B)].shape, device=DEV, generator=g).to(T.dtype)
    table = torch.randperm(B * nb, device=DEV, generator=g).view(B, nb).to(torch.int32)
    lens = [L - 29 * b for b in range(B)]
    row_bytes = 128 * K.element_size()
    assert Hkv * sum(lens) * row_bytes > 288 << 20
    ks = torch.tensor([k - b for b in range(B)], dtype=torch.int32, device=DEV)
    q = torch.randn((B, Hq, 128), device=DEV, generator=g)
    ctxs = []
    for filtered in (True, False):
        ctx = Lfps(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="f16" if dtype == "f16" else "bf16", max_seq_len=Lcap,
                   max_k=k, radius=r, k_fp8=kd == torch.float8_e4m3fn, v_fp8=vd == torch.float8_e4m3fn)
        ctx.lfps_set_filter(filtered)
        ctxs.append(ctx)
    prev = None
    for t in range(3):                                            # t = 0: the exact Top-k, then two steps (the second filtered)
        seq = torch.tensor([n + t for n in lens], dtype=torch.int32, device=DEV)
        res = []
        for ctx in ctxs:
            kv = ctx.paged_kv_view(K, V, table, seq) if page else ctx.kv_view(K, V, seq)
            idx = torch.full((B, Hq, k), -5, dtype=torch.int32, device=DEV)
            sc = torch.full((B, Hq, k), -5.0, device=DEV)
            out = torch.zeros((B, Hq, 128), device=DEV)
            if t == 0:
                ctx.lfps_exact_topk(q, kv, ks, idx, sc)
            else:
                ctx.lfps_step(q, kv, prev, ks, idx, out, sc)
                cnt = torch.zeros((B, Hkv), dtype=torch.int32, device=DEV)
                ctx.lfps_copy_cand_count(cnt)
                assert int(cnt.sum()) * row_bytes > 256 << 20
            res.append((idx, sc, out))
        for x, y, name in zip(*res, ("index", "score", "output")):
            assert torch.equal(x, y), (name, t, int((x != y).sum()))
        prev = res[0][0]
        q = q + 0.02 * torch.randn((B, Hq, 128), device=DEV, generator=g)
    assert ctxs[0].lfps_poll_rescored() == 0                      # the filtered passes decided, not their fall-back
    for ctx in ctxs:
        ctx.close()


# one query (stored dot products) and the most that are read past the caches, one more; against each request on its own, whose
# keys fit the cache: other sums of the exponentials, so entries agree to the 2e-5 of a table entry, not bit for bit
@pytest.mark.parametrize("dtype,page,B,L,Hq,Hkv,s", [
    ("bf16", 0, 5, 35007, 32, 8, 1), ("bf16", 16, 3, 70001, 16, 8, 4), ("f16", 64, 5, 33331, 8, 8, 8),
    ("fp8", 0, 8, 33007, 32, 8, 1), ("fp8", 16, 8, 33011, 16, 8, 3), ("bf16", 0, 4, 33007, 32, 8, 9)])
def test_tables_from_streamed_keys(dtype, page, B, L, Hq, Hkv, s):
    from paper_2506_15704_amd.binding import Lfps
    g = torch.Generator(device=DEV)
    g.manual_seed(L + s)
    kd = {"bf16": torch.bfloat16, "f16": torch.float16, "fp8": torch.float8_e4m3fn}[dtype]
    Lcap = L + 3
    nb = -(-Lcap // page) if page else 1
    shape = (B * nb, Hkv, page, 128) if page else (B, Hkv, Lcap, 128)
    K = torch.empty(shape, dtype=kd, device=DEV)
    for i in range(0, shape[0], nb):
        K[i:i + nb] = torch.randn(K[i:i + nb].shape, device=DEV, generator=g).to(kd)
    V = torch.zeros(shape, dtype=torch.float16 if dtype == "f16" else torch.bfloat16, device=DEV)
    assert B * Hkv * Lcap * 128 * K.element_size() > 256 << 20
    table = torch.randperm(B * nb, device=DEV, generator=g).view(B, nb).to(torch.int32)
    seq = torch.tensor([L - 127 * b for b in range(B)], dtype=torch.int32, device=DEV)
    q = 2 * torch.randn((s, B, Hq, 128), device=DEV, generator=g)

    def tables(lo, hi):
        ctx = Lfps(batch=hi - lo, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="f16" if dtype == "f16" else "bf16",
                   max_seq_len=Lcap, max_k=64, radius=1, k_fp8=dtype == "fp8", table_mode=True, table_decay=0.95, n_sink=4)
        n = seq[lo:hi].contiguous()
        kv = ctx.paged_kv_view(K, V, table[lo:hi].contiguous(), n) if page else ctx.kv_view(K[lo:hi], V[lo:hi], n)
        ctx.lfps_tables_init(q[:, lo:hi].contiguous(), kv)
        out = [torch.zeros((hi - lo, Hq, Lcap), dtype=torch.float64, device=DEV) for _ in range(2)]
        ctx.lfps_tables_export(*out, n)
        ctx.close()
        return out

    whole = tables(0, B)
    for b in range(B):
        for got, want in zip(whole, tables(b, b + 1)):
            assert float(want.abs().max()) > 0
            torch.testing.assert_close(got[b:b + 1], want, rtol=2e-5, atol=1e-12)


# every form of the kernels that ask how much is held; a request gives the same bits whatever the others hold
@pytest.mark.parametrize("dtype,page", [("bf16", 0), ("f16", 64), ("fp8k", 16), ("fp8kv", 0), ("fp8kv", 256), ("bf16", 16)])
@pytest.mark.parametrize("Hq,Hkv", [(8, 8), (16, 8), (32, 8)])
def test_full_attention_of_rows_read_once_equals_that_of_kept_rows(dtype, page, Hq, Hkv):
    from paper_2506_15704_amd.binding import Lfps
    g = torch.Generator(device=DEV)
    g.manual_seed(Hq + page)
    kd = {"bf16": torch.bfloat16, "f16": torch.float16}.get(dtype, torch.float8_e4m3fn)
    vd = torch.bfloat16 if dtype == "fp8k" else kd
    row = 128 * (torch.empty(0, dtype=kd).element_size() + torch.empty(0, dtype=vd).element_size())
    B = 3
    L = (340 << 20) // (B * Hkv * row) + 5
    nb = -(-L // page) if page else 1
    shape = (B * nb, Hkv, page, 128) if page else (B, Hkv, L, 128)
    K, V = (torch.empty(shape, dtype=d, device=DEV) for d in (kd, vd))
    for T in (K, V):
        for i in range(0, shape[0], nb):
            T[i:i + nb] = torch.randn(T[i:i + nb].shape, device=DEV, generator=g).to(T.dtype)
    table = torch.randperm(B * nb, device=DEV, generator=g).view(B, nb).to(torch.int32)
    q = torch.randn((B, Hq, 128), device=DEV, generator=g)
    ctx = Lfps(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="f16" if dtype == "f16" else "bf16", max_seq_len=L, max_k=1,
               radius=1, k_fp8=kd == torch.float8_e4m3fn, v_fp8=vd == torch.float8_e4m3fn)

    def attend(lens):
        seq = torch.tensor(lens, dtype=torch.int32, device=DEV)
        kv = ctx.paged_kv_view(K, V, table, seq) if page else ctx.kv_view(K, V, seq)
        out = torch.full((B, Hq, 128), 7.0, device=DEV)
        ctx.lfps_full_attn_decode(q, kv, out)
        return out

    lens = [L, L - 13, L - 1]
    assert sum(lens) * Hkv * row > 288 << 20
    whole = attend(lens)
    for b in range(B):
        few = attend([n if i == b else 1 for i, n in enumerate(lens)])
        assert torch.equal(few[b], whole[b]), b
    ctx.close()


@pytest.mark.parametrize("dtype,page", [("bf16", 0), ("f16", 64), ("fp8", 16), ("fp8", 0), ("bf16", 16)])
@pytest.mark.parametrize("Hq,s", [(32, 1), (32, 4), (8, 8), (16, 3)])
def test_tables_from_rows_read_once_equal_those_from_kept_rows(dtype, page, Hq, s):
    from paper_2506_15704_amd.binding import Lfps
    g = torch.Generator(device=DEV)
    g.manual_seed(Hq + s)
    kd = {"bf16": torch.bfloat16, "f16": torch.float16, "fp8": torch.float8_e4m3fn}[dtype]
    B, Hkv = 3, 8
    L = (300 << 20) // (B * Hkv * 128 * torch.empty(0, dtype=kd).element_size()) + 3
    nb = -(-L // page) if page else 1
    shape = (B * nb, Hkv, page, 128) if page else (B, Hkv, L, 128)
    K = torch.empty(shape, dtype=kd, device=DEV)
    for i in range(0, shape[0], nb):
        K[i:i + nb] = torch.randn(K[i:i + nb].shape, device=DEV, generator=g).to(kd)
    V = torch.zeros(shape, dtype=torch.float16 if dtype == "f16" else torch.bfloat16, device=DEV)
    table = torch.randperm(B * nb, device=DEV, generator=g).view(B, nb).to(torch.int32)
    q = 2 * torch.randn((s, B, Hq, 128), device=DEV, generator=g)
    ctx = Lfps(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="f16" if dtype == "f16" else "bf16", max_seq_len=L, max_k=64,
               radius=1, k_fp8=dtype == "fp8", table_mode=True, table_decay=0.95, n_sink=4)

    def tables(lens):
        seq = torch.tensor(lens, dtype=torch.int32, device=DEV)
        kv = ctx.paged_kv_view(K, V, table, seq) if page else ctx.kv_view(K, V, seq)
        ctx.lfps_tables_init(q, kv)
        out = [torch.zeros((B, Hq, L), dtype=torch.float64, device=DEV) for _ in range(2)]
        ctx.lfps_tables_export(*out, seq)
        return out

    lens = [L, L - 130, L - 1]
    whole = tables(lens)
    for b in range(B):
        few = tables([n if i == b else 200 for i, n in enumerate(lens)])
        for got, want in zip(whole, few):
            assert float(want[b].abs().max()) > 0
            assert torch.equal(got[b], want[b]), b
    ctx.close()
