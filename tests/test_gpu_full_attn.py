"""Full attention at the edges of its tiles (32 rows a wave, 16 in fp32 and without grouping), splits and groupings, with scores that are not finite:
against softmax and sum in fp64."""
import pytest
import torch

from tests.harness import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32", "fp8k", "fp8kv"])
@pytest.mark.parametrize("Hq,Hkv,lens,page", [
    (4, 1, [1, 31, 32, 33], 0), (8, 4, [64, 127, 129, 0], 16), (4, 4, [255, 256, 257, 15], 0), (16, 4, [511, 513, 17, 1030], 64),
    (4, 4, [1, 16, 17, 1030], 16), (2, 2, [63, 64, 65, 2113], 0)])
def test_full_attention_against_fp64(dtype, Hq, Hkv, lens, page):
    from paper_2506_15704_amd.binding import Lfps
    g = torch.Generator(device=DEV)
    g.manual_seed(Hq * 100 + max(lens))
    kd = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}.get(dtype, torch.float8_e4m3fn)
    vd = torch.bfloat16 if dtype == "fp8k" else kd
    B, Lcap, G = len(lens), max(lens), Hq // Hkv
    nb = -(-Lcap // page) if page else 1
    K, V = (torch.randn((B, Hkv, nb * page if page else Lcap, 128), device=DEV, generator=g).to(d) for d in (kd, vd))
    ctx = Lfps(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, kv_dtype=dtype if dtype in ("f16", "f32") else "bf16", max_seq_len=Lcap,
               max_k=1, radius=1, k_fp8=kd == torch.float8_e4m3fn, v_fp8=vd == torch.float8_e4m3fn)
    seq = torch.tensor(lens, dtype=torch.int32, device=DEV)
    if page:
        table = torch.randperm(B * nb, device=DEV, generator=g).view(B, nb)
        pools = []
        for T in (K, V):
            raw = T.view(torch.uint8) if T.element_size() == 1 else T
            blocks = raw.view(B, Hkv, nb, page, 128).permute(0, 2, 1, 3, 4).reshape(B * nb, Hkv, page, 128)
            pool = torch.zeros_like(blocks)
            pool[table.flatten()] = blocks
            pools.append(pool.view(T.dtype) if T.element_size() == 1 else pool)
        kv = ctx.paged_kv_view(*pools, table.to(torch.int32), seq)
    else:
        kv = ctx.kv_view(K, V, seq)
    q = 2.0 * torch.randn((B, Hq, 128), device=DEV, generator=g)
    out = torch.full((B, Hq, 128), 7.0, device=DEV)
    ctx.lfps_full_attn_decode(q, kv, out)
    for b, n in enumerate(lens):
        for h in range(Hq):
            if n == 0:
                assert torch.equal(out[b, h], torch.zeros_like(out[b, h]))
                continue
            k, v = K[b, h // G, :n].double(), V[b, h // G, :n].double()
            ref = torch.softmax(k @ q[b, h].double() / 128 ** 0.5, 0) @ v
            # fp32 dot products of scores up to 10 (1e-6), weights to the same, sums of up to 1030 terms
            assert float((out[b, h].double() - ref).abs().max()) <= 2e-5 * max(1.0, float(ref.abs().max())), (b, h)
    ctx.close()


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("Hkv", [2, 4, 8])
def test_rows_that_score_minus_infinity_weigh_nothing(dtype, Hkv):
    """Keys of -inf in one channel (positive there in every query): rows of weight 0, whole tiles of them among the others; a
    query beyond the fp16 range is no special case."""
    from paper_2506_15704_amd.binding import Lfps
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    dt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[dtype]
    L = 900
    K, V = (torch.randn((1, Hkv, L, 128), device=DEV, generator=g).to(dt) for _ in range(2))
    dead = torch.zeros(L, dtype=torch.bool, device=DEV)
    dead[:300] = True
    dead[400::3] = True
    K[:, :, :, 5] = 0
    K[:, :, dead, 5] = float("-inf")
    q = torch.randn((1, 8, 128), device=DEV, generator=g)
    q[..., 5] = 1e5
    ctx = Lfps(batch=1, n_q_heads=8, n_kv_heads=Hkv, kv_dtype=dtype, max_seq_len=L, max_k=1, radius=1)
    out = torch.zeros((1, 8, 128), device=DEV)
    ctx.lfps_full_attn_decode(q, ctx.kv_view(K, V, torch.tensor([L], dtype=torch.int32, device=DEV)), out)
    for h in range(8):
        k, v = K[0, h * Hkv // 8, ~dead].double(), V[0, h * Hkv // 8, ~dead].double()
        ref = torch.softmax(k @ q[0, h].double() / 128 ** 0.5, 0) @ v
        assert float((out[0, h].double() - ref).abs().max()) <= 2e-5
    ctx.close()
