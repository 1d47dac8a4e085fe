"""Candidates and scores in one kernel (chained steps of up to a million rows): at the edges of its ranges and pieces, from
the Top-k of the step before and from the table flags, against an unfiltered context, which takes other kernels.  (Larger contexts:
tests/test_wide_ranges.py.)  And the separate kernels, which the same steps take with a candidate capacity below the bound, as here."""
import pytest
import torch

from tests.harness import DEV

pytestmark = pytest.mark.gpu


def _pair(**kw):
    from paper_2506_15704_amd.binding import Lfps
    a, b = Lfps(**kw), Lfps(**kw)
    b.lfps_set_filter(False)
    return a, b


def _cache(B, Hkv, Lcap, dtype, page, g):
    dt = {"bf16": torch.bfloat16, "f16": torch.float16, "fp8": torch.bfloat16}[dtype]
    K, V = (torch.randn((B, Hkv, Lcap, 128), device=DEV, generator=g) for _ in range(2))
    K, V = K.to(torch.float8_e4m3fn) if dtype == "fp8" else K.to(dt), V.to(dt)
    if not page:
        return K, V, None
    nb = -(-Lcap // page)
    table = torch.randperm(B * nb, device=DEV, generator=g).view(B, nb)
    pool = []
    for x in (K, V):
        raw = torch.zeros((B, Hkv, nb * page, 128), dtype=x.dtype, device=DEV).view(torch.uint8)
        raw[:, :, :Lcap] = x.view(torch.uint8)
        p = torch.empty((B * nb, Hkv, page) + raw.shape[3:], dtype=torch.uint8, device=DEV)
        p[table.view(-1)] = raw.view(B, Hkv, nb, page, -1).transpose(1, 2).reshape(p.shape)
        pool.append(p.view(x.dtype))
    return pool[0], pool[1], table.to(torch.int32)


def _view(ctx, cache, seq):
    K, V, table = cache
    return ctx.kv_view(K, V, seq) if table is None else ctx.paged_kv_view(K, V, table, seq)


# lengths around multiples of a range (512, 1024), a quarter of it and a word; rows of prev_topk with and without 16-byte
# alignment (k % 4), more than 2048 entries per head, radius 0 and one wider than a range, sinks and recents across ranges
@pytest.mark.parametrize("B,Hq,Hkv,L,k,r,n_recent,n_sink,dtype,page", [
    (1, 4, 1, 1, 1, 0, 1, 0, "bf16", 0), (1, 4, 1, 511, 20, 2, 1, 0, "bf16", 0), (2, 8, 2, 1021, 33, 4, 0, 0, "bf16", 0),
    (1, 4, 4, 2047, 64, 3, 600, 700, "bf16", 0), (3, 8, 4, 3071, 63, 1, 1, 4, "f16", 16),
    (1, 8, 2, 12000, 2500, 1, 1, 0, "bf16", 0), (2, 4, 1, 1500, 10, 5000, 1, 0, "bf16", 0),
    (1, 32, 8, 40000, 500, 4, 1, 0, "bf16", 64), (5, 16, 8, 20000, 300, 2, 65, 2, "fp8", 0), (4, 32, 8, 30001, 90, 0, 1, 0, "fp8", 16)])
def test_memoryless_steps(B, Hq, Hkv, L, k, r, n_recent, n_sink, dtype, page):
    g = torch.Generator(device=DEV)
    g.manual_seed(L * 7 + k)
    Lcap = L + 6
    cache = _cache(B, Hkv, Lcap, dtype, page, g)
    a, b = _pair(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="bf16" if dtype == "fp8" else dtype, k_fp8=dtype == "fp8",
                 max_seq_len=Lcap, max_k=k, radius=r, n_recent=n_recent, n_sink=n_sink)
    lens = [max(1, L - 515 * i) for i in range(B)]
    ks = torch.tensor([max(1, min(k, n) - i) for i, n in enumerate(lens)], dtype=torch.int32, device=DEV)
    q = torch.randn((B, Hq, 128), device=DEV, generator=g)
    prev = torch.full((B, Hq, k), -1, dtype=torch.int32, device=DEV)
    a.lfps_exact_topk(q, _view(a, cache, torch.tensor(lens, dtype=torch.int32, device=DEV)), ks, prev)
    for t in range(1, 6):
        # slowly changing queries; then a useless history: every head takes the unfiltered pass from the bitmap
        q = q * 0.02 if t == 4 else q + 0.1 * torch.randn((B, Hq, 128), device=DEV, generator=g)
        if t == 3:      # a caller's list: unsorted, doubled, with entries that are no rows
            prev = prev.flip(2).contiguous()
            prev[:, :, ::7] = prev[:, :, :1].clone()
            for at, entry in ((3, -7), (5, 2**31 - 1), (6, L + 5), (8, -2**31)):
                prev[:, :, at::23] = entry
        seq = torch.tensor([n + t for n in lens], dtype=torch.int32, device=DEV)
        res = []
        for ctx in (a, b):
            idx = torch.full((B, Hq, k), -5, dtype=torch.int32, device=DEV)
            sc, out = torch.full((B, Hq, k), -5.0, device=DEV), torch.full((B, Hq, 128), -5.0, device=DEV)
            cnt = torch.full((B, Hkv), -5, dtype=torch.int32, device=DEV)
            ctx.lfps_step(q, _view(ctx, cache, seq), prev, ks, idx, out, sc)
            ctx.lfps_copy_cand_count(cnt)
            assert ctx.lfps_poll_status() == 0
            res.append((idx, sc, out, cnt))
        for x, y, name in zip(*res, ("index", "score", "output", "candidate count")):
            assert torch.equal(x, y), (name, t, int((x != y).sum()))
        prev = res[0][0]
    a.close()
    b.close()


@pytest.mark.parametrize("B,Hq,Hkv,L,k,r,n_sink,dtype,page", [
    (1, 4, 1, 100, 9, 1, 0, "bf16", 0), (2, 8, 2, 2047, 64, 1, 4, "bf16", 0), (2, 8, 4, 4099, 200, 30, 4, "f16", 64),
    (3, 8, 8, 9000, 100, 3, 4, "bf16", 16)])
def test_table_steps(B, Hq, Hkv, L, k, r, n_sink, dtype, page):
    g = torch.Generator(device=DEV)
    g.manual_seed(L + k)
    Lcap = L + 8
    cache = _cache(B, Hkv, Lcap, dtype, page, g)
    pair = _pair(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype=dtype, max_seq_len=Lcap, max_k=k, radius=r, n_sink=n_sink,
                 table_mode=True)
    lens = [max(1, L - 515 * i) for i in range(B)]
    ks = torch.tensor([min(k, n) for n in lens], dtype=torch.int32, device=DEV)
    q = 3 * torch.randn((B, Hq, 128), device=DEV, generator=g)
    for ctx in pair:
        ctx.lfps_tables_init(q[None].contiguous(), _view(ctx, cache, torch.tensor(lens, dtype=torch.int32, device=DEV)))
    for t in range(1, 6):
        q = q + 0.3 * torch.randn((B, Hq, 128), device=DEV, generator=g)
        seq = torch.tensor([n + t for n in lens], dtype=torch.int32, device=DEV)
        res = []
        for ctx in pair:
            idx = torch.full((B, Hq, k), -5, dtype=torch.int32, device=DEV)
            sc, out = torch.full((B, Hq, k), -5.0, device=DEV), torch.full((B, Hq, 128), -5.0, device=DEV)
            cnt = torch.full((B, Hkv), -5, dtype=torch.int32, device=DEV)
            ctx.lfps_table_step(q, _view(ctx, cache, seq), ks, idx, out, sc)
            ctx.lfps_copy_cand_count(cnt)
            res.append((idx, sc, out, cnt))
        for x, y, name in zip(*res, ("index", "score", "output", "candidate count")):
            assert torch.equal(x, y), (name, t, int((x != y).sum()))
    for ctx in pair:
        ctx.close()


# groups whose ranges of 1024 (2048 for the tables) rows would be more workgroups than the chip holds: five ranges of 1088, two of
# 2112 rows
def test_ranges_that_are_no_power_of_two():
    test_memoryless_steps(25, 8, 8, 5194, 60, 2, 1, 0, "bf16", 0)
    test_table_steps(43, 8, 8, 4100, 40, 2, 4, "f16", 0)


# more than 512 groups, which get one range each (of 5056 rows: 32 bits of the bitmap to a thread, threads past the range), or with
# four heads per group two of 2560
@pytest.mark.parametrize("Hq", [8, 32])
def test_one_range_per_group(Hq):
    test_table_steps(65, Hq, 8, 5000, 40, 2, 4, "bf16", 0)


@pytest.mark.parametrize("L,k", [(1200, 650), (3000, 1600)])
def test_a_budget_of_most_candidates_keeps_them_all(L, k):
    """A head whose budget takes more than half of its candidates remembers no threshold: other queries do not send it
    through the unfiltered pass."""
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    cache = _cache(1, 2, L, "bf16", 0, g)
    a, b = _pair(batch=1, n_q_heads=8, n_kv_heads=2, kv_dtype="bf16", max_seq_len=L, max_k=k, radius=0)
    seq, ks = (torch.tensor([x], dtype=torch.int32, device=DEV) for x in (L, k))
    prev = torch.randperm(L, device=DEV, generator=g)[:k].sort().values.to(torch.int32).expand(1, 8, k).contiguous()
    for t in range(3):
        q = torch.randn((1, 8, 128), device=DEV, generator=g) * (1.0, 3.0, 0.1)[t]
        res = []
        for ctx in (a, b):
            idx, out = torch.zeros((1, 8, k), dtype=torch.int32, device=DEV), torch.zeros((1, 8, 128), device=DEV)
            ctx.lfps_step(q, ctx.kv_view(cache[0], cache[1], seq), prev, ks, idx, out)
            res.append((idx, out))
        assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
    assert a.lfps_poll_rescored() == 0
    a.close()
    b.close()


# 1024, 512 and 256 threads per head; one to a few dozen words of bitmap, so that most waves own none
@pytest.mark.parametrize("B,Hq,Hkv,L,k,r,page", [
    (1, 4, 1, 40, 2, 0, 0), (2, 8, 2, 130, 8, 1, 16), (4, 32, 8, 301, 16, 2, 0), (8, 64, 16, 97, 5, 1, 0),
    (17, 32, 8, 260, 12, 1, 64), (17, 32, 32, 700, 20, 3, 0)])
def test_every_head_left_short_in_a_short_context(B, Hq, Hkv, L, k, r, page):
    """Queries fifty times smaller than the step before: no score reaches the remembered threshold and every head scores the
    group's candidates from the bitmap."""
    g = torch.Generator(device=DEV)
    g.manual_seed(L + k)
    Lcap = L + 8
    cache = _cache(B, Hkv, Lcap, "bf16", page, g)
    a, b = _pair(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="bf16", max_seq_len=Lcap, max_k=k, radius=r)
    ks = torch.full((B,), k, dtype=torch.int32, device=DEV)
    prev = torch.randint(0, L, (B, Hq, k), device=DEV, generator=g).to(torch.int32)
    for t in range(1, 8):
        q = torch.randn((B, Hq, 128), device=DEV, generator=g) * (4.0 if t % 2 else 0.02)
        seq = torch.tensor([L - i % 3 + t for i in range(B)], dtype=torch.int32, device=DEV)
        res = []
        for ctx in (a, b):
            idx = torch.full((B, Hq, k), -5, dtype=torch.int32, device=DEV)
            sc, out = torch.full((B, Hq, k), -5.0, device=DEV), torch.full((B, Hq, 128), -5.0, device=DEV)
            cnt = torch.full((B, Hkv), -5, dtype=torch.int32, device=DEV)
            ctx.lfps_step(q, _view(ctx, cache, seq), prev, ks, idx, out, sc)
            ctx.lfps_copy_cand_count(cnt)
            res.append((idx, sc, out, cnt))
        for x, y, name in zip(*res, ("index", "score", "output", "candidate count")):
            assert torch.equal(x, y), (name, t, int((x != y).sum()))
        if t % 2 == 0:
            assert a.lfps_poll_rescored() > 0.9 * B * Hq, t
        else:
            a.lfps_poll_rescored()
    a.close()
    b.close()


def _capacity_below_the_bound(**kw):
    """One candidate less than the largest set there can be: the range kernel is not taken (its bitmap is not allocated)."""
    from paper_2506_15704_amd.binding import workspace_bytes
    kw = dict(dict(head_dim=128, n_recent=1, n_sink=0, table_mode=0, k_fp8=0), **kw)
    bound = kw["n_q_heads"] // kw["n_kv_heads"] * kw["max_k"] * (2 * kw["radius"] + 2) + kw["n_recent"] + kw["n_sink"]
    bound = kw["max_seq_len"] if kw["table_mode"] else min(bound, kw["max_seq_len"])
    kw["kv_dtype"] = {"f32": 0, "bf16": 1, "f16": 2}[kw["kv_dtype"]]
    with_range, without = (workspace_bytes(cand_cap=c, **kw) for c in (bound, bound - 1))
    assert with_range - without >= kw["batch"] * kw["n_kv_heads"] * -(-kw["max_seq_len"] // 32) * 4
    return bound - 1


# 384 groups of a few hundred rows (one wave's part crosses several groups), few groups of many rows (a group is cut into
# many parts), one tiny group; 1, 2 and 4 heads per group
@pytest.mark.parametrize("B,Hq,Hkv,L,k,r,dtype,page", [
    (48, 32, 8, 700, 24, 1, "bf16", 0), (48, 32, 8, 700, 24, 1, "fp8", 16), (24, 16, 8, 900, 40, 2, "f16", 16),
    (40, 8, 8, 650, 30, 3, "bf16", 0), (5, 16, 4, 9000, 300, 2, "bf16", 64), (3, 16, 8, 20011, 400, 3, "f16", 64),
    (2, 4, 4, 12000, 500, 2, "fp8", 0), (1, 4, 1, 70, 5, 0, "bf16", 0)])
def test_memoryless_steps_through_the_separate_kernels(B, Hq, Hkv, L, k, r, dtype, page):
    g = torch.Generator(device=DEV)
    g.manual_seed(L * 3 + k)
    Lcap = L + 6
    cache = _cache(B, Hkv, Lcap, dtype, page, g)
    cfg = dict(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="bf16" if dtype == "fp8" else dtype, k_fp8=dtype == "fp8",
               max_seq_len=Lcap, max_k=k, radius=r)
    a, b = _pair(cand_cap=_capacity_below_the_bound(**cfg), **cfg)
    lens = [max(1, L - 131 * i % L) for i in range(B)]
    ks = torch.tensor([max(1, min(k, n) - i % 3) for i, n in enumerate(lens)], dtype=torch.int32, device=DEV)
    q = torch.randn((B, Hq, 128), device=DEV, generator=g)
    prev = torch.full((B, Hq, k), -1, dtype=torch.int32, device=DEV)
    a.lfps_exact_topk(q, _view(a, cache, torch.tensor(lens, dtype=torch.int32, device=DEV)), ks, prev)
    for t in range(1, 6):          # the fourth leaves every head short
        q = q * 0.02 if t == 4 else q + 0.1 * torch.randn((B, Hq, 128), device=DEV, generator=g)
        seq = torch.tensor([n + t for n in lens], dtype=torch.int32, device=DEV)
        res = []
        for ctx in (a, b):
            idx = torch.full((B, Hq, k), -5, dtype=torch.int32, device=DEV)
            sc, out = torch.full((B, Hq, k), -5.0, device=DEV), torch.full((B, Hq, 128), -5.0, device=DEV)
            cnt = torch.full((B, Hkv), -5, dtype=torch.int32, device=DEV)
            ctx.lfps_step(q, _view(ctx, cache, seq), prev, ks, idx, out, sc)
            ctx.lfps_copy_cand_count(cnt)
            assert ctx.lfps_poll_status() == 0
            res.append((idx, sc, out, cnt))
        for x, y, name in zip(*res, ("index", "score", "output", "candidate count")):
            assert torch.equal(x, y), (name, t, int((x != y).sum()))
        rescored = a.lfps_poll_rescored()
        assert t != 4 or rescored > B * Hq // 2, rescored
        prev = res[0][0]
    a.close()
    b.close()


@pytest.mark.parametrize("B,Hq,Hkv,L,k,r,dtype,page", [
    (48, 32, 8, 700, 24, 1, "bf16", 0), (24, 16, 8, 900, 40, 2, "f16", 16), (3, 8, 8, 9000, 100, 3, "bf16", 16)])
def test_table_steps_through_the_separate_kernels(B, Hq, Hkv, L, k, r, dtype, page):
    g = torch.Generator(device=DEV)
    g.manual_seed(L + k)
    Lcap = L + 8
    cache = _cache(B, Hkv, Lcap, dtype, page, g)
    cfg = dict(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype=dtype, max_seq_len=Lcap, max_k=k, radius=r, n_sink=4)
    pair = _pair(cand_cap=_capacity_below_the_bound(table_mode=1, table_decay=0.95, table_a=0.2, **cfg), table_mode=True, **cfg)
    lens = [max(1, L - 131 * i % L) for i in range(B)]
    ks = torch.tensor([min(k, n) for n in lens], dtype=torch.int32, device=DEV)
    q = 3 * torch.randn((B, Hq, 128), device=DEV, generator=g)
    for ctx in pair:
        ctx.lfps_tables_init(q[None].contiguous(), _view(ctx, cache, torch.tensor(lens, dtype=torch.int32, device=DEV)))
    for t in range(1, 6):
        q = q + 0.3 * torch.randn((B, Hq, 128), device=DEV, generator=g)
        seq = torch.tensor([n + t for n in lens], dtype=torch.int32, device=DEV)
        res = []
        for ctx in pair:
            idx = torch.full((B, Hq, k), -5, dtype=torch.int32, device=DEV)
            sc, out = torch.full((B, Hq, k), -5.0, device=DEV), torch.full((B, Hq, 128), -5.0, device=DEV)
            cnt = torch.full((B, Hkv), -5, dtype=torch.int32, device=DEV)
            ctx.lfps_table_step(q, _view(ctx, cache, seq), ks, idx, out, sc)
            ctx.lfps_copy_cand_count(cnt)
            res.append((idx, sc, out, cnt))
        for x, y, name in zip(*res, ("index", "score", "output", "candidate count")):
            assert torch.equal(x, y), (name, t, int((x != y).sum()))
    for ctx in pair:
        ctx.close()


def test_scores_that_grow_do_not_overflow_the_list():
    """Few heads with a small budget but many candidates: of the rows that reach the threshold of a step with smaller scores there may be
    more than 512 threads can hold, and as many as 1024 can: no head is rescored."""
    L, k, r = 65536, 512, 20
    g = torch.Generator(device=DEV)
    g.manual_seed(9)
    cache = _cache(1, 8, L, "bf16", 0, g)
    a, b = _pair(batch=1, n_q_heads=32, n_kv_heads=8, kv_dtype="bf16", max_seq_len=L, max_k=k, radius=r)
    seq, ks = (torch.tensor([x], dtype=torch.int32, device=DEV) for x in (L, k))
    q = torch.randn((1, 32, 128), device=DEV, generator=g)
    idx = [torch.full((1, 32, k), -1, dtype=torch.int32, device=DEV) for _ in range(4)]
    sc, out = torch.zeros((1, 32, k), device=DEV), torch.zeros((2, 1, 32, 128), device=DEV)
    a.lfps_exact_topk(q, _view(a, cache, seq), ks, idx[0])
    a.lfps_step(q, _view(a, cache, seq), idx[0], ks, idx[1], out[0], sc)
    scores = 4 * torch.einsum("hgd,hnd->hgn", q.view(8, 4, 128), cache[0][0].float()) / 128 ** 0.5
    near = torch.zeros((8, L + 2 * r + 1), dtype=torch.bool, device=DEV)      # candidates: the windows of a group's heads
    for d in range(2 * r + 2):
        near.scatter_(1, idx[1].view(8, -1).long() + d, True)
    survivors = ((scores >= sc.min(dim=2).values.view(8, 4, 1) - 0.125) & near[:, None, r:L + r]).sum(dim=2)
    assert 8192 < int(survivors.min()) and int(survivors.max()) < 16384, (int(survivors.min()), int(survivors.max()))
    assert a.lfps_poll_rescored() in (0, 32)                                     # (the first step may have kept everything)
    for ctx, at in ((a, 2), (b, 3)):
        ctx.lfps_step(4 * q, _view(ctx, cache, seq), idx[1], ks, idx[at], out[at - 2])
    assert a.lfps_poll_rescored() == 0
    assert torch.equal(idx[2], idx[3]) and torch.equal(out[0], out[1])
    a.close()
    b.close()
