"""The work a program that decodes with this library has it do, as timed cases.

Five kinds of pass, all through the public binding:

  step      `steps` consecutive decode steps of one attention layer (`lfps_step`), each on the Top-k the step before
            it left; the context has a history, as everywhere but at the first token of a request.
  tables    a request in the paper's score-table form with the head-sparsity bypass: history forgotten, tables from
            `n_hist` prefill queries, then `steps` decode steps (`lfps_table_step_gated`).
  handover  what prefill hands to decode: the priors and the tables from the last `n_hist` queries, and the tables as
            true values (the checkpoint).
  exact     the exact Top-k that seeds a request's history, and the sparse attention over it.
  full      full attention.

A case says the shapes (B requests of L rows, or of L_lo..L rows each when L_lo > 0; Hq query heads over Hkv KV heads
of 128 channels), the budget (k rows, or k_frac of a request's length in multiples of 64), the radius, the cache
format (dtype f32 / bf16 / f16 / fp8kv = FP8 keys and values / fp8k = FP8 keys beside bf16 values) and the layout
(page = rows per block, 0 = contiguous).
"""
import math

import torch

from paper_2506_15704_amd.binding import Lfps

D = 128
DEV = "cuda:0"
N_SINK = 4            # leading rows whose keys lean far towards the queries
N_LOCAL = 6           # local rows of the head-sparsity test (the paper's number)
EPS = 0.85            # its threshold (the paper's number)
DRIFT = 0.1           # change of a query from one decode step to the next

BASE = {"kind": "step", "B": 1, "L": 0, "L_lo": 0, "Hq": 32, "Hkv": 8, "dtype": "bf16", "page": 0, "k": 0,
        "k_frac": 0.0, "r": 4, "steps": 1, "n_hist": 0}


def _case(name, **kw):
    return dict(BASE, name=name, **kw)


def listed():
    return [
        # One short request, fp32 cache, one token: a step is three small kernels and the call's host work.
        _case("step_b1_4k_f32", B=1, L=4096, dtype="f32", k=128, r=2, steps=1),
        # One interactive request of ordinary length: latency.
        _case("step_b1_32k_bf16", B=1, L=32768, k=1024, r=4, steps=4),
        # A small batch of the same: the ordinary serving case.
        _case("step_b8_32k_bf16", B=8, L=32768, k=1024, r=4, steps=4),
        # The largest configuration of the benchmark: long contexts, 8.6 GB of cache per layer.
        _case("step_b16_128k_bf16", B=16, L=131072, k=2048, r=4, steps=4),
        # Continuous batching: every request has its own length, the budget is 2 % of it, narrow windows.
        _case("step_b32_ragged_bf16", B=32, L=65536, L_lo=16384, k_frac=0.02, r=2, steps=4),
        # The serving cache of large deployments: FP8 keys and values in a pool of 16-row blocks.
        _case("step_b16_64k_fp8kv_paged", B=16, L=65536, dtype="fp8kv", page=16, k=1024, r=4, steps=4),
        # A few requests of odd lengths, fp16 cache, two heads per group, larger blocks.
        _case("step_b3_odd_f16_paged", B=3, L=20011, L_lo=3001, Hq=16, Hkv=8, dtype="f16", page=64, k_frac=0.02, r=3,
              steps=4),
        # The paper's own rule over a request's first sixteen tokens, at an ordinary batch.
        _case("tables_b8_32k_bf16", kind="tables", B=8, L=32768, k=1024, r=1, steps=16, n_hist=1),
        # A request arriving from prefill: priors and tables from its last 32 queries (the paper's number).
        _case("handover_b1_32k_bf16", kind="handover", B=1, L=32768, k=1024, r=1, n_hist=32),
        # The seed of one request's history.
        _case("exact_b1_32k_bf16", kind="exact", B=1, L=32768, k=1024),
        # The seed of a batch of long requests.
        _case("exact_b8_64k_bf16", kind="exact", B=8, L=65536, k=1024),
        # Full attention over a batch: layers that stay dense.
        _case("full_b8_32k_bf16", kind="full", B=8, L=32768, k=1024),
    ]


def _logint(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _key_bytes(c):
    return {"f32": 4, "bf16": 2, "f16": 2, "fp8kv": 1, "fp8k": 1}[c["dtype"]]


def _value_bytes(c):
    return {"f32": 4, "bf16": 2, "f16": 2, "fp8kv": 1, "fp8k": 2}[c["dtype"]]


def draw(rng):
    most = max(work(c)["bytes"] for c in listed())
    while True:
        c = dict(BASE)
        c["kind"] = rng.choice(["step"] * 6 + ["tables", "handover", "exact", "full"])
        c["B"] = _logint(rng, 1, 32)
        c["L"] = _logint(rng, 2000, 131072)
        if rng.random() < 0.4 and c["B"] > 1:
            c["L_lo"] = max(1000, int(c["L"] * rng.uniform(0.15, 0.8)))
        c["Hq"], c["Hkv"] = rng.choice([(32, 8)] * 5 + [(16, 8), (8, 8), (16, 4)])
        c["dtype"] = rng.choice(["bf16"] * 4 + ["f16", "fp8kv", "fp8k", "f32"])
        c["page"] = rng.choice([0, 0, 0, 16, 64, 256])
        c["r"] = rng.choice([1, 2, 3, 4])
        if c["L_lo"]:
            c["k_frac"] = round(rng.uniform(1 / 64, 1 / 32), 4)
        else:
            c["k"] = max(48, int(c["L"] * rng.uniform(1 / 64, 1 / 32)))
        c["steps"] = {"step": rng.choice([1, 2, 4]), "tables": rng.choice([4, 8, 16])}.get(c["kind"], 1)
        c["n_hist"] = {"tables": rng.choice([1, 4]), "handover": rng.choice([8, 16, 32])}.get(c["kind"], 0)
        if c["kind"] in ("tables", "handover") and c["B"] * c["L"] > 8 * 65536:
            continue
        rows = c["B"] * c["Hkv"] * c["L"] * D
        if rows * (_key_bytes(c) + _value_bytes(c)) <= 16 * 8 * 131072 * D * 4 and work(c)["bytes"] <= most:
            return c


def _lengths(c, g):
    """Rows of every request before the first decode step (host ints)."""
    if not c["L_lo"]:
        return [c["L"]] * c["B"]
    n = torch.randint(c["L_lo"], c["L"] + 1, (c["B"],), generator=g).tolist()
    n[0] = c["L"]
    return n


def _budgets(c, lens):
    if not c["k_frac"]:
        return [min(c["k"], n) for n in lens]
    return [max(64, 64 * round(c["k_frac"] * n / 64)) for n in lens]


def _rms(x):
    return x / x.square().mean(dim=-1, keepdim=True).sqrt()


class _State:
    pass


def prepare(case, seed):
    """The layer's cache, its queries, lengths and budgets, a context and (for decode steps) the Top-k of the step
    before.  Keys are noise plus a bias towards their group's query direction on the first rows (sinks), on fixed hot
    rows and on the newest rows; queries start near that direction and drift from step to step.  The score-table
    kinds have more and stronger hot rows: their rule is made for attention that concentrates."""
    c = case
    host = torch.Generator()
    host.manual_seed(int(seed))
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 11)
    B, Hq, Hkv = c["B"], c["Hq"], c["Hkv"]
    G = Hq // Hkv
    tables = c["kind"] in ("tables", "handover")
    lens = _lengths(c, host)
    budgets = _budgets(c, lens)
    T = c["steps"] + 1 if c["kind"] in ("step", "tables") else 0     # rows appended after the first
    Lcap, kmax = c["L"] + T, max(budgets)

    # ---- keys and values
    kd = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}.get(c["dtype"], torch.float8_e4m3fn)
    vd = torch.bfloat16 if c["dtype"] == "fp8k" else kd

    def noise(rows_shape, dtype):
        out = torch.empty(rows_shape, dtype=dtype, device=DEV)
        raw = torch.bfloat16 if dtype == torch.float8_e4m3fn else dtype
        for i in range(rows_shape[0]):
            out[i] = torch.randn(rows_shape[1:], dtype=raw, device=DEV, generator=g).to(dtype)
        return out

    u = _rms(torch.randn((B, Hkv, D), device=DEV, generator=g))
    uhat = u / u.norm(dim=-1, keepdim=True)
    if c["page"]:
        bs = c["page"]
        nb = -(-Lcap // bs)
        K, V = (noise((B, nb, Hkv, bs, D), d).view(B * nb, Hkv, bs, D) for d in (kd, vd))
        table = torch.randperm(B * nb, generator=host).view(B, nb).to(torch.int32).to(DEV)
    else:
        K, V = (noise((B, Hkv, Lcap, D), d) for d in (kd, vd))
    beta_hot, n_hot = (7.0, max(16, c["L"] // 341)) if tables else (2.0, 16)
    for b in range(B):
        n = lens[b]
        beta_sink = math.log(n) + 1.1 if tables else 8.0      # tables: the sink share is near the bypass threshold
        hot = N_SINK + torch.randperm(n - 64 - N_SINK, generator=host)[:n_hot]
        rows = torch.cat([torch.arange(N_SINK), hot, torch.arange(max(n - 64, 0), Lcap)]).to(DEV)
        beta = torch.cat([torch.full((N_SINK,), beta_sink), torch.full((n_hot,), beta_hot),
                          torch.full((Lcap - max(n - 64, 0),), 3.0)]).to(DEV)
        lean = torch.randn((Hkv, rows.numel(), D), device=DEV, generator=g) + beta[None, :, None] * uhat[b][:, None, :]
        if c["page"]:
            blk, off = table[b].long()[rows // c["page"]], rows % c["page"]
            at = (blk[None, :], torch.arange(Hkv, device=DEV)[:, None], off[None, :])
        else:
            at = (torch.full((1, 1), b, device=DEV), torch.arange(Hkv, device=DEV)[:, None], rows[None, :])
        if kd == torch.float8_e4m3fn:
            K.view(torch.uint8).index_put_(at, lean.to(kd).view(torch.uint8))
        else:
            K.index_put_(at, lean.to(kd))

    # ---- queries: the history of a request (most recent first for the tables), then its decode steps
    n_hist = c["n_hist"]
    q = _rms(u.repeat_interleave(G, dim=1) + 0.3 * torch.randn((B, Hq, D), device=DEV, generator=g))
    chain = [q]
    for _ in range(n_hist + T):
        q = _rms(q + DRIFT * torch.randn((B, Hq, D), device=DEV, generator=g))
        chain.append(q)
    s = _State()
    s.case = c
    s.q_hist = torch.stack(chain[:n_hist][::-1]).contiguous() if n_hist else None
    s.q = [x.contiguous() for x in chain[n_hist:]]

    # ---- context, views
    s.ctx = Lfps(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype={"fp8kv": "bf16", "fp8k": "bf16"}.get(c["dtype"], c["dtype"]),
                 max_seq_len=Lcap, max_k=kmax, radius=c["r"], n_sink=N_SINK if tables else 0, table_mode=tables,
                 k_fp8=c["dtype"] in ("fp8kv", "fp8k"), v_fp8=c["dtype"] == "fp8kv")
    s.seq = [torch.tensor([n + t for n in lens], dtype=torch.int32, device=DEV) for t in range(T + 1)]
    if c["page"]:
        s.kv = [s.ctx.paged_kv_view(K, V, table, n) for n in s.seq]
    else:
        s.kv = [s.ctx.kv_view(K, V, n) for n in s.seq]
    s.k = torch.tensor(budgets, dtype=torch.int32, device=DEV)
    s.topk = [torch.full((B, Hq, kmax), -1, dtype=torch.int32, device=DEV) for _ in range(c["steps"])]
    s.out = [torch.zeros((B, Hq, D), device=DEV) for _ in range(c["steps"])]
    if tables:
        s.kbar, s.vbar = (torch.zeros((B, Hkv, D), device=DEV) for _ in range(2))
        s.sigma2 = torch.zeros((B, Hq), device=DEV)
        if c["kind"] == "handover":
            s.ver, s.sla = (torch.zeros((B, Hq, Lcap), dtype=torch.float64, device=DEV) for _ in range(2))
        else:
            s.ctx.lfps_priors(s.q_hist[0], s.kv[0], s.kbar, s.vbar, s.sigma2)
    if c["kind"] == "exact":
        s.score = torch.zeros((B, Hq, kmax), device=DEV)
    if c["kind"] == "step":
        seed_topk = torch.full((B, Hq, kmax), -1, dtype=torch.int32, device=DEV)
        s.prev = torch.full_like(seed_topk, -1)
        s.ctx.lfps_exact_topk(s.q[0], s.kv[0], s.k, seed_topk)
        s.ctx.lfps_step(s.q[1], s.kv[1], seed_topk, s.k, s.prev, s.out[0])
    torch.cuda.synchronize()
    return s


def run(s):
    c, ctx = s.case, s.ctx
    if c["kind"] == "step":
        prev = s.prev
        for t in range(c["steps"]):
            ctx.lfps_step(s.q[t + 2], s.kv[t + 2], prev, s.k, s.topk[t], s.out[t])
            prev = s.topk[t]
        return s.out, s.topk
    if c["kind"] == "tables":
        ctx.lfps_reset_history()
        ctx.lfps_tables_init(s.q_hist, s.kv[0])
        for t in range(c["steps"]):
            ctx.lfps_table_step_gated(s.q[t + 1], s.kv[t + 1], s.k, s.kbar, s.vbar, s.sigma2, N_LOCAL, EPS, s.topk[t],
                                      s.out[t])
        return s.out, s.topk
    if c["kind"] == "handover":
        ctx.lfps_priors(s.q_hist[0], s.kv[0], s.kbar, s.vbar, s.sigma2)
        ctx.lfps_tables_init(s.q_hist, s.kv[0])
        ctx.lfps_tables_export(s.ver, s.sla, s.seq[0])
        return s.kbar, s.vbar, s.sigma2, s.ver, s.sla
    if c["kind"] == "exact":
        ctx.lfps_exact_topk(s.q[0], s.kv[0], s.k, s.topk[0], s.score)
        ctx.lfps_sparse_attn(s.q[0], s.kv[0], s.topk[0], s.score, s.k, s.out[0])
        return s.topk[0], s.out[0]
    ctx.lfps_full_attn_decode(s.q[0], s.kv[0], s.out[0])
    return s.out[0]


def _mean_rows(c):
    return c["B"] * (0.5 * (c["L_lo"] + c["L"]) if c["L_lo"] else c["L"])


def work(case):
    """Bytes and multiply-adds (two operations each) of one pass, from the sizes.  The heads of a group select partly
    the same rows: a group's union is taken as 1, 1.3 or 1.6 budgets for 1, 2 or 4 heads, and its candidates as what
    windows of 2 r + 2 rows around that many random rows cover.  The table rule's candidates are taken as 4 % of the
    rows."""
    c = case
    rows = _mean_rows(c)                                  # rows of all requests, per KV head
    Hq, Hkv = c["Hq"], c["Hkv"]
    G = Hq // Hkv
    n = rows / c["B"]
    k = c["k_frac"] * n if c["k_frac"] else c["k"]
    row_k, row_v = D * _key_bytes(c), D * _value_bytes(c)
    union = min(n, {1: 1.0, 2: 1.3, 4: 1.6}[G] * k)
    heads, groups = c["B"] * Hq, c["B"] * Hkv
    io = heads * D * 8                                    # query in, output row out
    if c["kind"] in ("step", "tables"):
        cand = n * (1 - math.exp(-union * (2 * c["r"] + 2) / n)) if c["kind"] == "step" else 0.04 * n
        one = groups * (cand * row_k + min(union, cand) * row_v) + heads * k * 8 + io
        flops = 2.0 * D * heads * (cand + min(k, cand))
        if c["kind"] == "tables":
            one += heads * n * 8 + heads * min(k, cand) * 16   # both tables read, the selected entries updated
            start = groups * n * row_k + heads * n * 8 + c["n_hist"] * io
            return {"bytes": c["steps"] * one + start, "flops": c["steps"] * flops + 2.0 * D * heads * n * c["n_hist"]}
        return {"bytes": c["steps"] * one, "flops": c["steps"] * flops}
    if c["kind"] == "handover":                           # K and V once, tables written once, read and exported once
        return {"bytes": groups * n * (row_k + row_v) + heads * n * (8 + 8 + 16) + c["n_hist"] * io,
                "flops": 2.0 * D * heads * n * c["n_hist"]}
    if c["kind"] == "exact":
        return {"bytes": groups * (n * row_k + union * row_v) + heads * k * 16 + io, "flops": 2.0 * D * heads * (n + k)}
    return {"bytes": groups * n * (row_k + row_v) + io, "flops": 4.0 * D * heads * n}


def tolerance(case):
    """Measured against the same passes in 64 bits, four times what they differed by.  Where rows are selected, two
    rows whose scores agree to the last bit of fp32 sums may change places at the cut: a swap moves the entries of one
    head's ascending list between them (0.26 % of all entries at 8 x 32K) and one row of the average (1e-4 of the
    outputs' norm, 9e-3 of their root mean square in single elements).  Without a selection only sums differ."""
    if case["kind"] in ("full", "handover"):
        return {"rel": 3e-6, "max": 1e-5}
    return {"rel": 4e-4, "max": 4e-2, "differ": 1e-2}
