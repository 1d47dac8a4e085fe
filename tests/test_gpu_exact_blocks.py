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
