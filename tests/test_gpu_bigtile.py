"""The big-tile GEMM (32 ab rows x 256 columns, ab = 2..5) at the edges of its tiles: one row
more or less than whole tiles, a last column tile of fewer than 256 columns, fewer K slices
than its pipeline is deep and numbers that its depth does not divide, accumulation; and its fused
RoPE / cache-write epilogue against the LDS-tiled kernel's (whole windows of 129 .. 159 rows run there):
both add the products of a K range in the same order, so the caches agree bit for bit. Also the
LDS-tiled kernel's 128-row tiles, which very tall outputs of few columns take. Each case asserts the
plan that it is there for."""
import pytest
import torch

import workloads
from helpers import dev
from plans import gemm_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,acc,ab", [
    (4000, 5120, 64, False, 5),      # whole tiles, one slice
    (3999, 5120, 128, True, 5),      # two slices, ragged rows, accumulate
    (2305, 5120, 192, False, 3),     # one row past a tile
    (2304, 2048, 4096, True, 3),     # whole tiles, accumulate
    (4000, 2100, 320, True, 5),      # ragged columns
    (3999, 2048, 320, True, 4),      # one row less than whole tiles, five slices, accumulate
    (3970, 2040, 64, False, 4),      # 2 rows in the last tile, ragged columns, one slice
    (641, 5121, 2048, False, 2),     # ragged rows and columns
    (130, 60001, 256, False, 5),     # few rows, many columns
    (66000, 128, 64, False, 0),      # 128-row LDS tiles: ragged rows, one slice
    (65409, 100, 192, True, 0),      # one row in the last tile, ragged columns, accumulate
])
def test_bigtile_gemm(molt_lib, M, N, K, acc, ab):
    print(f"case M={M} N={N} K={K} acc={acc} ab={ab}", flush=True)
    plan = gemm_plan(M, N, K)
    assert (plan.ab, plan.bm) == ((ab, plan.bm) if ab else (0, 128))
    g = torch.Generator(device="cuda").manual_seed(M + N)
    A = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    B = torch.randn(N, K, generator=g, device="cuda").bfloat16()
    C0 = torch.randn(M, N, generator=g, device="cuda")
    C = molt_lib.dense_gemm(A, B, C0.clone() if acc else None, accumulate=acc).double()
    c0 = C0.double() if acc else torch.zeros_like(C)
    # f32 sum of K + 1 terms in any order: (K + 1) 2^-24 of the sum of magnitudes
    bound = (K + 1) * 2.0 ** -24 * (A.abs().double() @ B.abs().double().T + c0.abs())
    assert bool(((C - (A.double() @ B.double().T + c0)).abs() <= bound).all())


@pytest.mark.parametrize("Hq,Hkv,n,ctx,small,ab", [
    (32, 4, 705, 37, 141, 2),    # 40 heads, ragged rows
    (27, 9, 1500, 0, 150, 3),    # 45 heads: the last column tile holds one head
    (32, 4, 3999, 5, 129, 4),    # 40 heads, ragged rows
    (27, 9, 3975, 0, 159, 4),    # 45 heads, 7 rows in the last tile
])
def test_rope_epilogue_matches_small_windows(molt_lib, Hq, Hkv, n, ctx, small, ab):
    print(f"case Hq={Hq} Hkv={Hkv} n={n} ctx={ctx} ab={ab}", flush=True)
    assert [gemm_plan(m, (Hq + 2 * Hkv) * 128, 512, 0, rope=True).ab for m in (n, small)] == [ab, 0]
    w = workloads.LAYER_BF16.scaled(name="bigtile_rope", batch=1, k=n - 1, d_model=512, n_q_heads=Hq,
                                    n_kv_heads=Hkv, n_experts=4, top_k=2, d_ff=128, ctx_lo=ctx, ctx_hi=ctx)
    layout = workloads.make_kv_layout(w, 3)
    lw = workloads.make_layer_weights(w, 3, 0)
    model = molt_lib.Model([{k: dev(v) for k, v in lw.items()}], n_q_heads=Hq, n_kv_heads=Hkv,
                           head_dim=128, top_k=2)
    x = torch.randn(n, 512, generator=torch.Generator().manual_seed(4))
    bt = dev(torch.from_numpy(layout.block_tables))
    caches = []
    for window in (n, small):
        kc, vc = (dev(c) for c in workloads.make_kv_cache(w, layout, 3, 0))
        rows = []
        for s in range(0, n, window):
            m = min(window, n - s)
            kv = molt_lib.KVCache([kc], [vc], bt, torch.tensor([ctx + s], dtype=torch.int32, device="cuda"))
            xs = dev(x[s:s + m].clone())
            molt_lib.decoder_forward(model, kv, 1, m - 1, xs)
            rows.append(xs)
        caches.append((kc, vc, torch.cat(rows)))
    assert torch.equal(caches[0][0], caches[1][0])
    assert torch.equal(caches[0][1], caches[1][1])
    # q (also written by the epilogue) shows in the layer's output; bf16 storage steps and
    # split-K orders downstream stay far inside 2e-2, a wrong rotation does not
    assert float((caches[0][2] - caches[1][2]).abs().max()) <= 2e-2
