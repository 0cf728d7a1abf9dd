"""Slots of the KV cache past a sequence's last token hold anything (a cache that is written slot by
slot is never initialised): attention with every such slot, and every block that no sequence uses, an
infinity or NaN, against the oracle on the clean cache. Up to 64 rows per query tile and more, both head
sizes, splits with empty and odd last blocks, prefill windows. Tolerance as for finite caches: scores and
16-bit probabilities in two parts leave less than 1e-3 at values of N(0, 1), the output is rounded to
bf16."""
import numpy as np
import pytest
import torch

import workloads
from oracle import attention as oattn, model as omodel
from helpers import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fill", [float("nan"), float("inf")])
@pytest.mark.parametrize("B,k,Hq,Hkv,D,lo,hi", [
    (3, 0, 8, 2, 128, 0, 40),          # 4 rows: one or two pairs
    (4, 4, 32, 4, 128, 14, 18),        # 40 rows, contexts around a block's end
    (2, 7, 8, 1, 64, 100, 900),        # 64 rows, head size 64, short splits
    (5, 2, 8, 1, 128, 1, 2500),        # ragged, splits of 32 blocks, some empty
    (3, 8, 8, 1, 128, 0, 30),          # 72 rows: two 16-row tiles per wavefront
    (2, 15, 16, 2, 64, 500, 1500),     # 128 rows, splits
    (1, 40, 8, 2, 128, 7, 7),          # windows of several query tiles, each with its own last key
    (3, 100, 8, 1, 128, 0, 60),
])
def test_tail(molt_lib, B, k, Hq, Hkv, D, lo, hi, fill):
    print(f"case B={B} k={k} Hq={Hq} Hkv={Hkv} D={D} ctx=[{lo},{hi}] fill={fill}", flush=True)
    w = workloads.LAYER_BF16.scaled(batch=B, k=k, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, ctx_lo=lo, ctx_hi=hi)
    layout = workloads.make_kv_layout(w, 17)
    kc, vc = workloads.make_kv_cache(w, layout, 17, 0)
    T = B * (k + 1)
    q = torch.randn(T, Hq, D, generator=workloads.rng(17, "q")).bfloat16()
    ref = oattn.paged_attention(omodel.widen_cache(host(q), "bf16"), omodel.widen_cache(host(kc), "bf16"),
                                omodel.widen_cache(host(vc), "bf16"), layout.block_tables,
                                layout.context_lens, k).reshape(T, -1)
    used = torch.zeros(kc.shape[0], 16, dtype=torch.bool)
    for b in range(B):
        p = np.arange(int(layout.context_lens[b]) + k + 1)
        used[torch.from_numpy(layout.block_tables[b, p // 16].astype(np.int64)), torch.from_numpy(p % 16)] = True
    kc = torch.where(used[:, None, :, None], kc, torch.full_like(kc, fill))
    vc = torch.where(used[:, None, None, :], vc, torch.full_like(vc, fill))
    out = molt_lib.paged_attention(dev(q), dev(kc), dev(vc), dev(torch.from_numpy(layout.block_tables)),
                                   dev(torch.from_numpy(layout.context_lens)), k).float().cpu().numpy()
    assert bool((np.abs(out - ref) <= np.abs(ref) * 2.0 ** -8 + 1e-3).all())
