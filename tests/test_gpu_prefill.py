"""The prefill hand-over (Eq. 4 from many queries, the priors) at the edges of its kernels' tiles, against the oracle.

Table entries are sums of up to s fp32 weights, each with a relative error of a few 2^-24 (exponential, normalisation,
rounding): rtol 2e-5 as in test_gpu_tables.  Means are fp32 roundings of sums of fp32 partial sums of at most a few
hundred unit-variance rows: atol 2e-6; the variance is relative to its own size: rel 2e-5."""
import numpy as np
import pytest
import torch

import gen
from gen import device as gen_device
from oracle import lfps_oracle as orc
from oracle import lfps_tables_oracle as tor
from tests.harness import DEV, DeviceCase, dev

pytestmark = pytest.mark.gpu


def _view(ctx, dc, seq, page):
    if not page:
        return ctx.kv_view(dc.K, dc.V, seq)
    Kp, Vp, table = gen_device.paginate(dc.K, dc.V, page, seed=3)
    return ctx.paged_kv_view(Kp, Vp, table, seq)


def _case(name, L, heads, fmt, B=2):
    kw = {"fp8": dict(k_dtype="fp8"), "fp8kv": dict(k_dtype="fp8", v_dtype="fp8")}.get(fmt, dict(kv_dtype=fmt))
    return DeviceCase(gen.tiny_spec(name, B=B, L=L, k=min(16, L), Hq=heads[0], Hkv=heads[1], n_hot=0 if L < 200 else 4,
                                    recency=min(16, L // 2), **kw))


# lengths around the 128-row tiles and the 1024 rows of a workgroup, shorter than the history and than the sinks;
# histories around the batch of 32 queries
@pytest.mark.parametrize("L,s,heads,fmt,page", [
    (127, 32, (8, 2), "bf16", 0), (128, 33, (8, 2), "bf16", 16), (129, 31, (8, 2), "fp8", 0), (1025, 5, (8, 2), "f16", 0),
    (1024, 65, (4, 2), "bf16", 0), (2111, 32, (4, 2), "fp8", 64), (385, 64, (2, 2), "f16", 16), (20, 32, (8, 2), "bf16", 0),
    (5, 3, (2, 2), "bf16", 0), (700, 32, (8, 2), "f32", 0)])
def test_tables_from_many_queries(L, s, heads, fmt, page):
    dc = _case("hist", L, heads, fmt)
    spec, case = dc.spec, dc.case
    n_sink, gamma = 4, 0.95
    ctx = dc.make_ctx(table_mode=True, table_decay=gamma, n_sink=n_sink)
    rng = np.random.default_rng(7)
    q = rng.standard_normal((s, spec.B, spec.Hq, spec.D)).astype(np.float32) * np.float32(1.5)
    # tables that held a longer sequence before: nothing of it may be left
    ctx.lfps_tables_init(dev(q[:2]), _view(ctx, dc, dc.seq_lens(spec.T), page))
    ctx.lfps_tables_init(dev(q), _view(ctx, dc, dc.seq_lens(0), page))
    ev = torch.zeros((spec.B, spec.Hq, case.Lcap), dtype=torch.float64, device=DEV)
    es = torch.zeros_like(ev)
    ctx.lfps_tables_export(ev, es, dc.seq_lens(spec.T))
    ev, es = ev.cpu().numpy(), es.cpu().numpy()
    G = spec.G
    for b, h in ((0, 0), (1, spec.Hq - 1), (1, G - 1)):
        K, _ = dc.group(b, h // G)
        n = int(case.seq_lens0[b])
        w = np.zeros((s, n))
        for j in range(1, s + 1):
            seen = n - j + 1
            if seen > n_sink:
                sc = orc.scores(q[j - 1, b, h], K[:seen])[n_sink:]
                e = np.exp(sc - sc.max())
                w[j - 1, n_sink:seen] = e / e.sum()
        ver, sla = tor.init_tables(w, gamma, n_sink)
        np.testing.assert_allclose(ev[b, h, :n], ver, rtol=2e-5, atol=1e-12)
        np.testing.assert_allclose(es[b, h, :n], sla, rtol=2e-5, atol=1e-12)
        assert not ev[b, h, n:].any() and not es[b, h, n:].any()
    # the statistics: candidates from them
    cand = torch.zeros((spec.B, spec.Hkv, ctx.cand_cap), dtype=torch.int32, device=DEV)
    cnt = torch.zeros((spec.B, spec.Hkv), dtype=torch.int32, device=DEV)
    ctx.lfps_table_candidates(dc.seq_lens(0), cand, cnt)
    n = int(case.seq_lens0[0])
    t64 = [(ev[0, h, :n], es[0, h, :n]) for h in range(G)]
    want = tor.group_candidates(t64, n, float(np.float32(0.2)), spec.r, 1, n_sink)
    got = cand[0, 0, : int(cnt[0, 0])].cpu().numpy()
    assert len(np.setxor1d(got, want)) <= n // 500        # entries within a rounding of a threshold
    ctx.close()


# ungrouped heads: one unit of sixteen queries (spans of sixteen rows, which all sixteen queries reach across), two, and both in
# turn; lengths around a span, a chunk of 128 rows and a workgroup
@pytest.mark.parametrize("L,s,fmt,page", [
    (17, 16, "bf16", 0), (127, 16, "bf16", 0), (129, 15, "fp8", 16), (1041, 9, "f16", 0), (2111, 16, "bf16", 64), (300, 17, "bf16", 0),
    (1024, 48, "fp8", 0), (640, 2, "bf16", 16)])
def test_tables_of_ungrouped_heads(L, s, fmt, page):
    test_tables_from_many_queries(L, s, (2, 2), fmt, page)


# one unit of grouped heads over FP8 keys (four queries of four heads, eight of two), and a last batch of one behind a full one
@pytest.mark.parametrize("L,s,heads,page", [
    (17, 4, (8, 2), 0), (127, 3, (8, 2), 16), (1041, 8, (4, 2), 0), (129, 5, (4, 2), 64), (2111, 4, (8, 2), 0), (640, 2, (8, 2), 16),
    (1025, 36, (8, 2), 0), (300, 40, (4, 2), 16)])
def test_tables_of_one_unit_over_fp8_keys(L, s, heads, page):
    test_tables_from_many_queries(L, s, heads, "fp8", page)


@pytest.mark.parametrize("L,heads,fmt,page,n_sink", [
    (255, (8, 2), "bf16", 0, 4), (257, (4, 2), "fp8kv", 16, 0), (1030, (2, 2), "fp8", 0, 4), (777, (8, 2), "f16", 64, 4),
    (513, (8, 2), "f32", 0, 1), (17, (8, 2), "bf16", 0, 4), (3, (8, 2), "bf16", 0, 4)])
def test_priors_at_split_edges(L, heads, fmt, page, n_sink):
    dc = _case("priors", L, heads, fmt)
    spec, case = dc.spec, dc.case
    ctx = dc.make_ctx(n_sink=n_sink)
    kbar = torch.full((spec.B, spec.Hkv, spec.D), 9.0, device=DEV)
    vbar = torch.full_like(kbar, 9.0)
    s2 = torch.full((spec.B, spec.Hq), 9.0, device=DEV)
    ctx.lfps_priors(dc.q(0), _view(ctx, dc, dc.seq_lens(0), page), kbar, vbar, s2)
    for b in range(spec.B):
        n = int(case.seq_lens0[b])
        for g in range(spec.Hkv):
            K, V = dc.group(b, g)
            for h in range(spec.G):
                if n <= n_sink:
                    ok, ov, os2 = np.zeros(spec.D), np.zeros(spec.D), 0.0
                else:
                    ok, ov, os2 = tor.priors(case.q[0, b, spec.G * g + h], K, V, n, n_sink)
                np.testing.assert_allclose(kbar[b, g].cpu().numpy(), ok, rtol=0, atol=2e-6)
                np.testing.assert_allclose(vbar[b, g].cpu().numpy(), ov, rtol=0, atol=2e-6)
                assert float(s2[b, spec.G * g + h]) == pytest.approx(os2, rel=2e-5, abs=1e-9)
    ctx.close()


# four partials a group merged by one workgroup (256 groups and more) and by five, sixteen, seventeen and 128 partials; requests with
# no rows, with fewer than there are parts, with all.  The bounds of the test above: 24-bit sums over n / 64 rows at most.
@pytest.mark.parametrize("B,Hq,Hkv,L", [(300, 1, 1, 70), (32, 32, 8, 300), (255, 2, 1, 513), (64, 4, 1, 4090), (61, 4, 1, 4353), (1, 8, 8, 32768)])
def test_priors_however_the_partials_are_merged(B, Hq, Hkv, L):
    from paper_2506_15704_amd.binding import Lfps
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    K, V = (torch.randn((B, Hkv, L, 128), device=DEV, generator=g).to(torch.bfloat16) for _ in range(2))
    q = torch.randn((B, Hq, 128), device=DEV, generator=g)
    lens = [max(0, L - 17 * b) for b in range(B)]
    ctx = Lfps(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, max_seq_len=L, max_k=4, radius=1, n_sink=3)
    kbar, vbar = (torch.full((B, Hkv, 128), 9.0, device=DEV) for _ in range(2))
    s2 = torch.full((B, Hq), 9.0, device=DEV)
    ctx.lfps_priors(q, ctx.kv_view(K, V, torch.tensor(lens, dtype=torch.int32, device=DEV)), kbar, vbar, s2)
    G = Hq // Hkv
    for b in range(B):
        rows = K[b, :, 3:lens[b]].double(), V[b, :, 3:lens[b]].double()
        if lens[b] <= 3:
            assert not (kbar[b].any() or vbar[b].any() or s2[b].any())
            continue
        for got, x in ((kbar, rows[0]), (vbar, rows[1])):
            torch.testing.assert_close(got[b].double(), x.mean(1), rtol=0, atol=2e-6)
        qb = q[b].double().view(Hkv, G, 128)
        want = (rows[0] @ qb.transpose(1, 2).contiguous() / 128**0.5).var(1, unbiased=False) / qb.square().sum(-1)
        torch.testing.assert_close(s2[b].double().view(Hkv, G), want, rtol=2e-5, atol=1e-9)
    ctx.close()


# one query (from stored dot products), one batch of queries, two; rows in whole 128-row tiles and in the ones cut by the
# sinks and by the end
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("s", [1, 5, 33])
@pytest.mark.parametrize("bad,value", [((4, 130, 131, 255, 600, 699), -np.inf), ((200,), np.nan), ((5, 690), np.nan),
                                       ((300,), np.inf)])
def test_tables_where_scores_are_not_finite(dtype, s, bad, value):
    """A row that scores -inf weighs nothing.  Where a score is NaN or +inf the softmax has no value: the entries of that row
    are NaN and the query adds nothing elsewhere."""
    from paper_2506_15704_amd.binding import Lfps
    L, n_sink, gamma = 700, 4, 0.95
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    g = torch.Generator(device=DEV)
    g.manual_seed(s)
    K = torch.randn((1, 1, L + 8, 128), device=DEV, generator=g).to(dt)
    q = torch.randn((s, 1, 2, 128), device=DEV, generator=g).to(torch.bfloat16).float()   # (whole in one term of the split)
    q[..., :2] = 2.0
    for i in bad:
        K[0, 0, i] = 0
        K[0, 0, i, :2] = {-np.inf: -3e38, np.inf: 3e38}.get(value, value)                  # 2 * -3e38 - ... = -inf in fp32
    ctx = Lfps(batch=1, n_q_heads=2, n_kv_heads=1, kv_dtype=dtype, max_seq_len=L + 8, max_k=16, radius=1, n_sink=n_sink,
               table_mode=True, table_decay=gamma)
    seq = torch.tensor([L], dtype=torch.int32, device=DEV)
    ctx.lfps_tables_init(q.contiguous(), ctx.kv_view(K, K, seq))
    ver, sla = (torch.zeros((1, 2, L + 8), dtype=torch.float64, device=DEV) for _ in range(2))
    ctx.lfps_tables_export(ver, sla, seq)
    for h in range(2):
        w = np.zeros((s, L))
        for j in range(1, s + 1):
            seen = L - j + 1
            sc = orc.scores(q[j - 1, 0, h].cpu().numpy(), K[0, 0, :seen].float().cpu().numpy())[n_sink:]
            at = np.array([i - n_sink for i in bad if i < seen], dtype=int)
            sc[at] = -np.inf
            w[j - 1, n_sink:seen] = np.exp(sc - sc.max()) / np.exp(sc - sc.max()).sum()
            if value != -np.inf and len(at):
                w[j - 1] = 0
                w[j - 1, at + n_sink] = np.nan
        want = tor.init_tables(w, gamma, n_sink)
        for got, ref in zip((ver, sla), want):
            np.testing.assert_allclose(got[0, h, :L].cpu().numpy(), ref, rtol=2e-5, atol=1e-12)
    ctx.close()


@pytest.mark.parametrize("B", [1, 64, 128])
def test_means_hold_their_accuracy_for_many_groups(B):
    """The sums of a group's rows: 64 chains of fp32 additions, added in fp64, at most, whatever the number of groups.  All
    requests share their rows (one table), so that many groups are small in memory.  Held to the RMS error of such chains,
    simulated (over 2048 means: known to 2 %), with 25 % to spare; chains of n / 32 rows have twice that error."""
    from paper_2506_15704_amd.binding import Lfps
    L, page, Hkv = 8192, 256, 8
    g = torch.Generator(device=DEV)
    g.manual_seed(B)
    K, V = (0.5 + 0.3 * torch.randn((L // page, Hkv, page, 128), device=DEV, generator=g) for _ in range(2))
    table = torch.arange(L // page, device=DEV, dtype=torch.int32).expand(B, L // page).contiguous()
    ctx = Lfps(batch=B, n_q_heads=Hkv, n_kv_heads=Hkv, kv_dtype="f32", max_seq_len=L, max_k=16, radius=1)
    q = torch.randn((B, Hkv, 128), device=DEV, generator=g)
    kbar, vbar = torch.zeros((B, Hkv, 128), device=DEV), torch.zeros((B, Hkv, 128), device=DEV)
    seq = torch.full((B,), L, dtype=torch.int32, device=DEV)
    ctx.lfps_priors(q, ctx.paged_kv_view(K, V, table, seq), kbar, vbar, torch.zeros((B, Hkv), device=DEV))
    errs, sims = [], []
    for X, got in ((K, kbar), (V, vbar)):
        x = X.transpose(1, 2).reshape(L, Hkv, 128).cpu().numpy()
        mean = x.mean(axis=0, dtype=np.float64)
        chains = np.cumsum(x.reshape(L // 64, 64, Hkv, 128), axis=0, dtype=np.float32)[-1]     # row i in chain i % 64
        sims.append((chains.astype(np.float64).sum(axis=0) / L).astype(np.float32) - mean)
        errs.append(got[B - 1].cpu().numpy() - mean)
    rms = lambda e: float(np.sqrt(np.mean(np.square(np.stack(e)))))
    assert rms(errs) <= 1.25 * rms(sims), (rms(errs), rms(sims))
    ctx.close()


@pytest.mark.parametrize("s", [1, 6])
def test_tables_of_many_groups_are_those_of_few(s):
    """320 KV groups, one workgroup each: every request's tables as in a context of that request alone, in which each group is
    cut into several.  The sums of exponentials are in fp64, so the weights differ by a rounding: 2 units of 2^-24 each."""
    from paper_2506_15704_amd.binding import Lfps
    B, Hkv, L = 40, 8, 2100
    g = torch.Generator(device=DEV)
    g.manual_seed(s)
    K = torch.randn((B, Hkv, L, 128), device=DEV, generator=g).to(torch.bfloat16)
    q = torch.randn((s, B, Hkv, 128), device=DEV, generator=g)
    lens = [L - 41 * b for b in range(B)]

    def tables(rows):
        n = len(rows)
        ctx = Lfps(batch=n, n_q_heads=Hkv, n_kv_heads=Hkv, kv_dtype="bf16", max_seq_len=L, max_k=16, radius=1, n_sink=4,
                   table_mode=True)
        seq = torch.tensor([lens[b] for b in rows], dtype=torch.int32, device=DEV)
        Kr = K[rows].contiguous()
        ctx.lfps_tables_init(q[:, rows].contiguous(), ctx.kv_view(Kr, Kr, seq))
        out = torch.zeros((2, n, Hkv, L), dtype=torch.float64, device=DEV)
        ctx.lfps_tables_export(out[0], out[1], seq)
        torch.cuda.synchronize()
        ctx.close()
        return out

    many = tables(list(range(B)))
    for b in (0, 17, B - 1):
        few = tables([b])
        assert (many[:, b] - few[:, 0]).abs().max() <= 2.0**-23 * few.abs().max()
        assert (few > 0).any()


# Several queries in one pass: histories around the four queries of a quad and the units of four, eight and sixteen queries that
# make other kernels, lengths around the 64- and 128-row chunks, the 32 rows before a span and one chunk per workgroup
@pytest.mark.parametrize("L,s,heads,fmt,page", [
    (63, 2, (8, 2), "bf16", 0), (65, 4, (8, 2), "fp8", 16), (129, 8, (8, 2), "bf16", 0), (191, 9, (8, 2), "f16", 0),
    (257, 16, (8, 2), "bf16", 64), (2049, 17, (8, 2), "fp8", 0), (96, 8, (4, 2), "bf16", 16), (321, 15, (4, 2), "f16", 0),
    (1500, 30, (4, 2), "bf16", 0), (161, 3, (2, 2), "f16", 16), (290, 16, (2, 2), "fp8", 0), (4100, 32, (2, 2), "bf16", 0),
    (33, 32, (2, 2), "bf16", 0), (640, 40, (8, 2), "bf16", 256)])
def test_tables_at_the_edges_of_chunks_and_units(L, s, heads, fmt, page):
    test_tables_from_many_queries(L, s, heads, fmt, page)
