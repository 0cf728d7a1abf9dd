"""GPU parity of the attention of query tiles with more than 64 rows (one or two 16-row tiles
per wavefront) at its edges: 5, 6, 7 and 8 tiles, partial tiles, both head sizes, one key pair
and fewer, contexts at block ends, splits (also empty ones), and prefill windows whose last
query tile is short. The output is a float32 sum rounded to bf16 (2^-9 of its value); scores
and 16-bit probabilities in two parts leave less than 1e-3 at values of N(0, 1)."""
import numpy as np
import pytest
import torch

import workloads
from oracle import attention as oattn, model as omodel
from helpers import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,k,Hq,Hkv,D,lo,hi", [
    (3, 8, 8, 1, 128, 0, 30),          # 72 rows: 5 tiles, the last half full; one or two pairs
    (2, 10, 16, 2, 128, 15, 17),       # 88 rows: 6 tiles, contexts around a block's end
    (2, 24, 6, 2, 64, 40, 700),        # 75 rows of 3 heads a group, head size 64
    (2, 15, 16, 2, 128, 500, 1500),    # 128 rows: 8 full tiles, splits
    (5, 12, 8, 1, 64, 1, 2500),        # 104 rows: 7 tiles, ragged with empty splits
    (1, 32, 8, 2, 128, 7, 7),          # 33 positions of 4 heads: 128 rows and a tile of 4
    (3, 100, 8, 1, 128, 0, 60),        # 7 query tiles, the last with 5 positions
])
def test_rows(molt_lib, B, k, Hq, Hkv, D, lo, hi):
    print(f"case B={B} k={k} Hq={Hq} Hkv={Hkv} D={D} ctx=[{lo},{hi}]", flush=True)
    w = workloads.LAYER_BF16.scaled(batch=B, k=k, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, ctx_lo=lo, ctx_hi=hi)
    layout = workloads.make_kv_layout(w, 11)
    kc, vc = workloads.make_kv_cache(w, layout, 11, 0)
    T = B * (k + 1)
    q = torch.randn(T, Hq, D, generator=workloads.rng(11, "q")).bfloat16()
    ref = oattn.paged_attention(omodel.widen_cache(host(q), "bf16"), omodel.widen_cache(host(kc), "bf16"),
                                omodel.widen_cache(host(vc), "bf16"), layout.block_tables,
                                layout.context_lens, k).reshape(T, -1)
    out = molt_lib.paged_attention(dev(q), dev(kc), dev(vc), dev(torch.from_numpy(layout.block_tables)),
                                   dev(torch.from_numpy(layout.context_lens)), k).float().cpu().numpy()
    assert bool((np.abs(out - ref) <= np.abs(ref) * 2.0 ** -8 + 1e-3).all())
