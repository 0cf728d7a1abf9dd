"""GPU parity of the f32 model's kernels at the edges of their tiles: the f32 MFMA GEMM (32 x
32 tiles, K slices of 32 split over 8 wavefronts: fewer slices than wavefronts, remainders,
ragged rows and columns), the f32 expert GEMMs over several row tiles per expert, and the
f32 attention (64-key chunks over 4 wavefronts, both head sizes). A sum of n products in f32
is within n 2^-24 of the sum of magnitudes whatever the order, which gives the bounds."""
import pytest
import torch

import workloads
from oracle import attention as oattn
from helpers import dev, host, max_abs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,acc", [
    (1, 32, 32, False),       # one slice: 7 wavefronts without work
    (16, 100, 224, False),    # 7 slices, ragged columns
    (33, 96, 288, True),      # 9 slices, two row tiles, accumulate
    (65, 65, 1056, False),    # 33 slices
])
def test_f32_gemm(molt_lib, M, N, K, acc):
    print(f"case M={M} N={N} K={K} acc={acc}", flush=True)
    g = torch.Generator().manual_seed(M + N + K)
    A, B, C0 = torch.randn(M, K, generator=g), torch.randn(N, K, generator=g), torch.randn(M, N, generator=g)
    C = molt_lib.dense_gemm(A.cuda(), B.cuda(), C0.clone().cuda() if acc else None, accumulate=acc).cpu().double()
    c0 = C0.double() if acc else torch.zeros(M, N, dtype=torch.float64)
    bound = (K + 1) * 2.0 ** -24 * (A.abs().double() @ B.abs().double().T + c0.abs())
    assert bool(((C - (A.double() @ B.double().T + c0)).abs() <= bound).all())


@pytest.mark.parametrize("T,d,E,K,F", [(1, 64, 3, 1, 64), (75, 128, 4, 2, 192), (130, 64, 2, 2, 64)])
def test_f32_moe(molt_lib, T, d, E, K, F):
    print(f"case T={T} d={d} E={E} K={K} F={F}", flush=True)
    g = torch.Generator().manual_seed(T)
    x = torch.randn(T, d, generator=g)
    wr, wgu, wd = (torch.randn(E, d, generator=g), 0.1 * torch.randn(E, 2 * F, d, generator=g),
                   0.1 * torch.randn(E, d, F, generator=g))
    ids = torch.rand(T, E, generator=g).topk(K, -1).indices.int()
    out = molt_lib.moe_layer(dev(x), dev(wr), dev(wgu), dev(wd), K, replay_ids=dev(ids)).cpu().double()
    X, W = x.double(), wr.double()
    p = torch.softmax((X @ W.T).gather(1, ids.long()), -1)
    ref = torch.zeros(T, d, dtype=torch.float64)
    for t in range(T):
        for j in range(K):
            e = int(ids[t, j])
            v = wgu[e].double() @ X[t]
            ref[t] += p[t, j] * (wd[e].double() @ (v[:F] * torch.sigmoid(v[:F]) * v[F:]))
    # the hardware exp2 and reciprocal of SiLU are good to ~1e-6 relative
    assert max_abs(out.numpy(), ref.numpy()) <= 1e-5 * float(ref.abs().max() + 1)


@pytest.mark.parametrize("D,k,lo,hi", [(64, 0, 0, 0), (64, 2, 15, 17), (128, 1, 60, 66), (128, 3, 250, 700)])
def test_f32_attention(molt_lib, D, k, lo, hi):
    print(f"case D={D} k={k} ctx=[{lo},{hi}]", flush=True)
    B, Hq, Hkv = 3, 6, 2
    w = workloads.LAYER_BF16.scaled(batch=B, k=k, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, ctx_lo=lo,
                                    ctx_hi=hi, dtype="f32")
    layout = workloads.make_kv_layout(w, 5)
    kc, vc = workloads.make_kv_cache(w, layout, 5, 0)
    q = torch.randn(B * (k + 1), Hq, D, generator=workloads.rng(5, "q"))
    ref = oattn.paged_attention(host(q), host(kc), host(vc), layout.block_tables, layout.context_lens, k)
    # slots past a sequence's last key hold anything, also NaN
    for b in range(B):
        n = int(layout.context_lens[b]) + k + 1
        blk = int(layout.block_tables[b, (n - 1) // 16])
        if n % 16:
            kc[blk, :, n % 16:] = float("nan")
            vc[blk, :, :, n % 16:] = float("nan")
    out = molt_lib.paged_attention(dev(q), dev(kc), dev(vc), dev(torch.from_numpy(layout.block_tables)),
                                   dev(torch.from_numpy(layout.context_lens)), k)
    assert max_abs(out.cpu().numpy(), ref.reshape(B * (k + 1), -1)) <= 1e-5


@pytest.mark.parametrize("lo,hi", [(0, 0), (70, 70), (300, 300)])
def test_f32_attention_scores_of_any_size(molt_lib, lo, hi):
    """Finite scores far below -1e30 (queries and keys of 1e17): the softmax depends on their
    differences only. Each query of -1e17 e_0 meets keys of first component 1e17 + small, so that
    scores are about -1e33 and one key's is the largest by far: the output is that key's value."""
    print(f"case ctx=[{lo},{hi}]", flush=True)
    B, k, Hq, Hkv, D = 2, 1, 2, 1, 64
    w = workloads.LAYER_BF16.scaled(batch=B, k=k, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, ctx_lo=lo,
                                    ctx_hi=hi, dtype="f32")
    layout = workloads.make_kv_layout(w, 6)
    kc, vc = workloads.make_kv_cache(w, layout, 6, 0)
    kc[:] = 0
    kc[..., 0] = 1e17
    best = {}
    for b in range(B):
        p = (lo + 1) // 2 if lo else 0
        blk = int(layout.block_tables[b, p // 16])
        kc[blk, 0, p % 16, 0] = 0.9e17
        best[b] = vc[blk, 0, :, p % 16]
    q = torch.zeros(B * (k + 1), Hq, D)
    q[..., 0] = -1e17
    out = molt_lib.paged_attention(dev(q), dev(kc), dev(vc), dev(torch.from_numpy(layout.block_tables)),
                                   dev(torch.from_numpy(layout.context_lens)), k).cpu().view(B, k + 1, Hq, D)
    for b in range(B):
        assert bool((out[b] == best[b]).all())
