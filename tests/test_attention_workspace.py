"""Workspaces of calls with attention. Few sequences of short tables take finer splits of the key range
than a larger batch does, which need more workspace; one that holds the splits of 32 blocks is accepted
as well, so that a workspace sized for other arguments serves (results then come from those splits).
On the CPU: what is refused; on the GPU: what is accepted, against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2607_21653_amd as molt
import workloads
from oracle import attention as oattn, model as omodel
from helpers import dev, host, model_from

WORKSPACE = -3
# B, k, Hq, Hkv, D, blocks of the longest table: where the finer splits need more
FINE = [(1, 4, 32, 4, 128, 512), (16, 4, 32, 4, 128, 32), (2, 0, 8, 1, 64, 20), (3, 8, 8, 1, 128, 100),
        (1, 40, 8, 2, 128, 40)]


def _coarse(B, k, Hq, Hkv, D, mb):
    """Bytes of the partial results with splits of at least 32 blocks (0: one split)."""
    G, kp1 = Hq // Hkv, k + 1
    tq = kp1 if G * kp1 <= 128 else 128 // G
    units = B * Hkv * -(-kp1 // tq)
    s = max(1, min(-(-512 // units), -(-mb // 32)))
    bps = -(-(-(-mb // s)) // 8) * 8
    s = -(-mb // bps)
    if s == 1:
        return 0
    rows, al = B * kp1 * Hq * s, lambda n: -(-n // 256) * 256
    return al(rows * D * 4) + rows * 8 + 256


@pytest.mark.parametrize("case", FINE)
def test_refused_below_the_coarse_splits(case):
    L = molt.load()
    B, k, Hq, Hkv, D, mb = case
    coarse, full = _coarse(*case), L.molt_paged_attention_workspace_size(*case)
    assert full > coarse
    if coarse:
        p = ctypes.c_void_p(0x1000)
        for ws, n in ((p, coarse - 1), (None, full)):
            assert L.molt_paged_attention(p, p, p, p, p, B, k, Hq, Hkv, D, mb, 1, p, ws, n, None) == WORKSPACE


@pytest.mark.parametrize("B,k,Hq,Hkv,D", [(1, 4, 32, 4, 128), (3, 0, 8, 1, 64), (2, 60, 16, 4, 128)])
def test_size_holds_the_coarse_splits(B, k, Hq, Hkv, D):
    for mb in range(1, 2049):
        args = (B, k, Hq, Hkv, D, mb)
        assert molt.load().molt_paged_attention_workspace_size(*args) >= _coarse(*args), mb


@pytest.mark.gpu
@pytest.mark.parametrize("case", FINE)
def test_coarse_splits_are_accepted(molt_lib, case):
    print(f"case {case}", flush=True)
    B, k, Hq, Hkv, D, mb = case
    hi = 16 * mb - k - 1
    w = workloads.LAYER_BF16.scaled(batch=B, k=k, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, ctx_lo=hi // 2, ctx_hi=hi)
    layout = workloads.make_kv_layout(w, 13)
    bt = np.full((B, mb), -1, np.int32)
    n = min(mb, layout.block_tables.shape[1])
    bt[:, :n] = layout.block_tables[:, :n]
    kc, vc = workloads.make_kv_cache(w, layout, 13, 0)
    T = B * (k + 1)
    q = torch.randn(T, Hq, D, generator=workloads.rng(13, "q")).bfloat16()
    ref = oattn.paged_attention(omodel.widen_cache(host(q), "bf16"), omodel.widen_cache(host(kc), "bf16"),
                                omodel.widen_cache(host(vc), "bf16"), bt, layout.context_lens, k).reshape(T, -1)
    qd, kd, vd = dev(q), dev(kc), dev(vc)
    btd, ctx = dev(torch.from_numpy(bt)), dev(torch.from_numpy(layout.context_lens))
    L = molt_lib.load()
    for size in (_coarse(*case), L.molt_paged_attention_workspace_size(*case)):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda") if size else None
        out = torch.empty(T, Hq * D, dtype=torch.bfloat16, device="cuda")
        p = lambda t: None if t is None else t.data_ptr()
        assert L.molt_paged_attention(p(qd), p(kd), p(vd), p(btd), p(ctx), B, k, Hq, Hkv, D, mb, 1, p(out), p(ws),
                                      size, torch.cuda.current_stream().cuda_stream) == 0
        got = out.float().cpu().numpy()
        assert bool((np.abs(got - ref) <= np.abs(ref) * 2.0 ** -8 + 1e-3).all()), size


@pytest.mark.gpu
def test_decoder_with_a_coarse_workspace(molt_lib):
    """A decoder call whose workspace lacks the finer splits' part: the same layer, other split sums."""
    B, k, mb = 2, 2, 64
    w = workloads.LAYER_BF16.scaled(batch=B, k=k, d_model=256, n_q_heads=8, n_kv_heads=2, head_dim=128, n_experts=4,
                                    top_k=2, d_ff=128, ctx_lo=900, ctx_hi=16 * mb - k - 1)
    layout = workloads.make_kv_layout(w, 4)
    model = model_from(w, [workloads.make_layer_weights(w, 4, 0)], None, molt_lib)
    x0 = torch.randn(B * (k + 1), 256, generator=workloads.rng(4, "x")).cuda()
    mb = layout.block_tables.shape[1]
    full = molt_lib.decoder_workspace_size(model, B, k, mb)
    args = (B, k, 8, 2, 128, mb)
    less = full - (molt_lib.load().molt_paged_attention_workspace_size(*args) - _coarse(*args)) + 256
    assert less < full
    out = []
    for size in (full, less):
        kc, vc = workloads.make_kv_cache(w, layout, 4, 0)
        kv = molt_lib.KVCache([dev(kc)], [dev(vc)], dev(torch.from_numpy(layout.block_tables)),
                              dev(torch.from_numpy(layout.context_lens)))
        ws = torch.empty(size + 4096, dtype=torch.uint8, device="cuda").fill_(0x5a)
        x = x0.clone()
        assert molt_lib.load().molt_decoder_forward(
            ctypes.byref(model.struct), ctypes.byref(kv.struct), B, k, x.data_ptr(), None, ws.data_ptr(), size,
            torch.cuda.current_stream().cuda_stream) == 0
        assert bool((ws[size:] == 0x5a).all())          # the call stays inside what it was given
        out.append(x)
    assert float((out[0] - out[1]).abs().max()) <= 2e-2
