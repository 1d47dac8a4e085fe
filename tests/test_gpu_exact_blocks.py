"""The exact Top-k of rows whose scoring pass leaves the largest score of every 16: bit for bit against the select over the same
scores given as a candidate list, which other tests hold against the oracle."""
import pytest
import torch

from tests.harness import DEV

pytestmark = pytest.mark.gpu


# one block more than 512; the largest budgets that are selected from blocks and the next ones (select_takes_tops); a thread with
# several blocks; rows past a multiple of 16 and of 64; 2, 4, 8 and 16 blocks per thread of the choice, and more than that
@pytest.mark.parametrize("L,k", [(8193, 1), (8193, 513), (8193, 514), (8207, 300), (32768, 1024), (32769, 2047), (65537, 4097),
                                 (131073, 1500), (262144, 100), (262145, 100), (8193, 496), (8193, 497), (32768, 1760),
                                 (32768, 1761), (32769, 1984), (32769, 1985), (131073, 6528), (131073, 6529), (262144, 8448),
                                 (262144, 8449)])
@pytest.mark.parametrize("values", ["normal", "ties", "equal", "runs", "special"])
def test_select_from_block_maxima(L, k, values):
    from paper_2506_15704_amd.binding import Lfps
    g = torch.Generator(device=DEV)
    g.manual_seed(L + k)
    Hq, Hkv = 4, 1
    K = torch.randn((1, Hkv, L, 128), device=DEV, generator=g)
    q = torch.randn((1, Hq, 128), device=DEV, generator=g)
    if values == "ties":
        K = K[:, :, :7][:, :, torch.randint(0, 7, (L,), device=DEV, generator=g)].contiguous()
    if values == "equal":
        K[:] = K[:, :, :1]
    if values == "runs":                     # long runs of high scores: whole blocks reach the cut
        K[:, :, L // 3:L // 3 + 2 * k] += 2 * q[:, :1, None, 0]
        K[:, :, : min(16 * k, L // 2)] += 0.5 * q[0, 0]
    if values == "special":                  # scores that are not finite, one row each and a whole block
        K[0, 0, L // 2, 3] = float("inf")
        K[0, 0, 77, 5] = float("nan")
        K[0, 0, 4096:4112, 9] = float("-inf")
    K = K.to(torch.bfloat16)
    ctx = Lfps(batch=1, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="bf16", max_seq_len=L + 3, max_k=k, radius=1, cand_cap=L)
    K = torch.nn.functional.pad(K, (0, 0, 0, 3))
    seq, kk = (torch.tensor([x], dtype=torch.int32, device=DEV) for x in (L, k))
    kv = ctx.kv_view(K, K, seq)
    idx = [torch.full((1, Hq, k), -5, dtype=torch.int32, device=DEV) for _ in range(2)]
    sc = [torch.full((1, Hq, k), -5.0, device=DEV) for _ in range(2)]
    ctx.lfps_exact_topk(q, kv, kk, idx[0], sc[0])
    cand = torch.arange(ctx.cand_cap, dtype=torch.int32, device=DEV).view(1, 1, -1).contiguous()
    ctx.lfps_score_topk(q, kv, cand, torch.tensor([[L]], dtype=torch.int32, device=DEV), kk, idx[1], sc[1])
    assert torch.equal(idx[0], idx[1])
    assert torch.equal(sc[0].view(torch.int32), sc[1].view(torch.int32))
    ctx.close()


# requests of different lengths (one whose row is selected from all scores), groups with lanes that compute maxima and store none, the
# other cache formats and pages; the last budget lies past the line
@pytest.mark.parametrize("dtype,page", [("bf16", 16), ("f16", 0), ("f16", 64), ("fp8", 0), ("fp8", 16)])
@pytest.mark.parametrize("Hq,Hkv", [(8, 8), (8, 4), (16, 4)])
def test_block_maxima_of_a_ragged_batch(dtype, page, Hq, Hkv):
    from paper_2506_15704_amd.binding import Lfps
    g = torch.Generator(device=DEV)
    g.manual_seed(Hq + page)
    lens, budgets = [33001, 8191, 20015, 16400], [1500, 700, 1, 1020]
    B, L, k = len(lens), max(lens) + 2, max(budgets)
    kd = {"bf16": torch.bfloat16, "f16": torch.float16, "fp8": torch.float8_e4m3fn}[dtype]
    nb = -(-L // page) if page else 1
    shape = (B * nb, Hkv, page, 128) if page else (B, Hkv, L, 128)
    K = torch.randn(shape, device=DEV, generator=g).to(kd)
    V = torch.zeros(shape, dtype=torch.float16 if dtype == "f16" else torch.bfloat16, device=DEV)
    q = torch.randn((B, Hq, 128), device=DEV, generator=g)
    ctx = Lfps(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype="f16" if dtype == "f16" else "bf16", max_seq_len=L, max_k=k,
               radius=1, cand_cap=L, k_fp8=dtype == "fp8")
    seq, ks = (torch.tensor(x, dtype=torch.int32, device=DEV) for x in (lens, budgets))
    table = torch.randperm(B * nb, device=DEV, generator=g).view(B, nb).to(torch.int32)
    kv = ctx.paged_kv_view(K, V, table, seq) if page else ctx.kv_view(K, V, seq)
    idx = [torch.full((B, Hq, k), -5, dtype=torch.int32, device=DEV) for _ in range(2)]
    sc = [torch.full((B, Hq, k), -5.0, device=DEV) for _ in range(2)]
    ctx.lfps_exact_topk(q, kv, ks, idx[0], sc[0])
    cand = torch.arange(ctx.cand_cap, dtype=torch.int32, device=DEV).repeat(B, Hkv, 1)
    ctx.lfps_score_topk(q, kv, cand, seq[:, None].repeat(1, Hkv), ks, idx[1], sc[1])
    for b, kb in enumerate(budgets):
        assert int(idx[0][b, :, :kb].min()) >= 0
        assert torch.equal(idx[0][b, :, :kb], idx[1][b, :, :kb])
        assert torch.equal(sc[0][b, :, :kb].view(torch.int32), sc[1][b, :, :kb].view(torch.int32))
    ctx.close()
