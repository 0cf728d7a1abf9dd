"""Calls with few rows: the few-row QKV projection with its RoPE / cache-write epilogue (32- and
64-row tiles, K slices that 8 wavefronts do not divide, odd head counts), attention of a few short sequences over many short splits, and top-K over every split
count of the router GEMM."""
import numpy as np
import pytest
import torch

import workloads
from oracle import attention as oattn, model as omodel
from helpers import dev, host, max_abs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,k,Hq,Hkv,d,ctx", [
    (1, 0, 2, 1, 128, 0),         # one row, two K slices
    (1, 30, 4, 2, 640, 5),        # 31 rows, 10 slices
    (11, 2, 3, 1, 2048, 100),     # 33 rows
    (64, 0, 8, 2, 1152, 31),      # 64 rows, 18 slices
    (13, 4, 32, 4, 2048, 700),    # 65 rows: two row tiles
    (32, 3, 6, 3, 2688, 40),      # 128 rows, 42 slices
])
def test_qkv_few_rows(molt_lib, B, k, Hq, Hkv, d, ctx):
    print(f"case B={B} k={k} Hq={Hq} Hkv={Hkv} d={d} ctx={ctx}", flush=True)
    T, D = B * (k + 1), 128
    w = workloads.LAYER_BF16.scaled(name="few", batch=B, k=k, d_model=d, n_q_heads=Hq, n_kv_heads=Hkv,
                                    n_experts=2, top_k=1, d_ff=64, ctx_lo=ctx, ctx_hi=ctx)
    layout = workloads.make_kv_layout(w, 3)
    lw = workloads.make_layer_weights(w, 3, 0)
    model = molt_lib.Model([{n: dev(v) for n, v in lw.items()}], n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, top_k=1)
    kc, vc = workloads.make_kv_cache(w, layout, 3, 0)
    bt2 = layout.block_tables
    xs = torch.randn(T, d, generator=torch.Generator().manual_seed(1))
    gk, gv = dev(kc), dev(vc)
    kv = molt_lib.KVCache([gk], [gv], dev(torch.from_numpy(bt2)), dev(torch.from_numpy(layout.context_lens)))
    molt_lib.decoder_forward(model, kv, B, k, dev(xs.clone()))
    n = len(xs)
    y = (xs.double() / (xs.double().square().mean(1, keepdim=True) + 1e-6).sqrt()).bfloat16().double()
    wq = lw["w_qkv"].double()
    qkv = (y @ wq.T).view(n, Hq + 2 * Hkv, D)
    mag = (y.abs() @ wq.abs().T).view(n, Hq + 2 * Hkv, D)
    pos = torch.from_numpy(np.concatenate([np.arange(ctx, ctx + k + 1)] * B)).double()
    ang = pos[:, None] * 1.0e6 ** (-2.0 * torch.arange(64).double() / D)
    co, si = ang.cos()[:, None], ang.sin()[:, None]
    kk, kmag = qkv[:, Hq:Hq + Hkv], mag[:, Hq:Hq + Hkv]
    kr = torch.cat([kk[..., :64] * co - kk[..., 64:] * si, kk[..., 64:] * co + kk[..., :64] * si], -1)
    kmag = kmag[..., :64] + kmag[..., 64:]
    kmag = torch.cat([kmag, kmag], -1)
    new = torch.zeros(kc.shape[0], 16, dtype=torch.bool)
    gk, gv = gk.cpu().double(), gv.cpu().double()
    # a bf16 step where the sum sits at a rounding boundary (the norm's own roundings among them)
    for t in range(n):
        b, p = t // (k + 1), ctx + t % (k + 1)
        blk, sl = int(bt2[b, p // 16]), p % 16
        new[blk, sl] = True
        assert bool(((gk[blk, :, sl] - kr[t]).abs() <= kr[t].abs() * 2.0 ** -8 + 2.0 ** -8 * 0.02 * 8 + 2.0 ** -18 * kmag[t]).all())
        v = qkv[t, Hq + Hkv:]
        assert bool(((gv[blk, :, :, sl] - v).abs() <= v.abs() * 2.0 ** -8 + 2.0 ** -8 * 0.02 * 8 + 2.0 ** -18 * mag[t, Hq + Hkv:]).all())
    # every other slot is untouched
    assert bool((gk.permute(0, 2, 1, 3)[~new] == kc.double().permute(0, 2, 1, 3)[~new]).all())
    assert bool((gv.permute(0, 3, 1, 2)[~new] == vc.double().permute(0, 3, 1, 2)[~new]).all())


@pytest.mark.parametrize("B,k,Hq,Hkv,D,lo,hi", [
    (1, 4, 32, 4, 128, 1500, 1500),    # 12 splits of 8 blocks
    (1, 0, 8, 1, 64, 130, 130),        # two splits, the second of one block
    (2, 8, 16, 2, 128, 3, 2000),       # 72 rows, most splits of one sequence empty
    (1, 4, 8, 1, 128, 65000, 65000),   # 128 splits
])
def test_attention_few_sequences(molt_lib, B, k, Hq, Hkv, D, lo, hi):
    print(f"case B={B} k={k} Hq={Hq} Hkv={Hkv} D={D} ctx=[{lo},{hi}]", flush=True)
    w = workloads.LAYER_BF16.scaled(batch=B, k=k, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, ctx_lo=lo, ctx_hi=hi)
    layout = workloads.make_kv_layout(w, 12)
    kc, vc = workloads.make_kv_cache(w, layout, 12, 0)
    T = B * (k + 1)
    q = torch.randn(T, Hq, D, generator=workloads.rng(12, "q")).bfloat16()
    ref = oattn.paged_attention(omodel.widen_cache(host(q), "bf16"), omodel.widen_cache(host(kc), "bf16"),
                                omodel.widen_cache(host(vc), "bf16"), layout.block_tables,
                                layout.context_lens, k).reshape(T, -1)
    out = molt_lib.paged_attention(dev(q), dev(kc), dev(vc), dev(torch.from_numpy(layout.block_tables)),
                                   dev(torch.from_numpy(layout.context_lens)), k).float().cpu().numpy()
    assert bool((np.abs(out - ref) <= np.abs(ref) * 2.0 ** -8 + 1e-3).all())


@pytest.mark.parametrize("T,d", [(3, 2048), (3, 512), (3, 256), (3, 128), (700, 2048), (3, 8192)])
def test_topk_split_counts(molt_lib, T, d):
    """Exact integers: whatever the number of split-K partials, ids and weights are the same."""
    E, K = 130, 5
    g = np.random.Generator(np.random.Philox(d + T))
    x = torch.from_numpy(g.integers(-2, 3, (T, d)).astype(np.float32)).bfloat16()
    wr = torch.from_numpy((g.integers(-1, 2, (E, d)) / 16.0).astype(np.float32)).bfloat16()
    z = torch.zeros(E, 128, d, dtype=torch.bfloat16, device="cuda")
    _, ids, wts, *_ = molt_lib.moe_layer(dev(x), dev(wr), z, torch.zeros(E, d, 64, dtype=torch.bfloat16, device="cuda"),
                                         K, want_routing=True)
    logits = (x.double() @ wr.double().T).numpy()
    order = np.lexsort((np.broadcast_to(np.arange(E), logits.shape), -logits), axis=1)[:, :K]
    assert (ids.cpu().numpy() == order).all()
    sel = np.take_along_axis(logits, order, 1)
    ex = np.exp(sel - sel[:, :1])
    assert max_abs(wts.cpu().numpy(), ex / ex.sum(1, keepdims=True)) <= 1e-6
