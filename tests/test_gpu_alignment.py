"""bf16 arrays that start at any element: KV caches and expert rows that are not aligned to 16 bytes take
another way into LDS (attention of more than 64 query rows, the big-tile expert GEMM), with the same
arithmetic: the same bits as from aligned arrays."""
import pytest
import torch

import workloads
from helpers import dev
from plans import BF16, moe_plan

pytestmark = pytest.mark.gpu


def _shifted(t, n):
    """A copy of t that starts n elements past an aligned address."""
    buf = torch.empty(t.numel() + n, dtype=t.dtype, device="cuda")
    v = buf[n:].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 == n * t.element_size() % 16
    return v


@pytest.mark.parametrize("kn,vn", [(1, 4), (0, 7), (4, 0)])
@pytest.mark.parametrize("B,k,Hq,Hkv,D,lo,hi", [
    (3, 4, 8, 2, 128, 5, 200),         # 20 rows: copied through registers anyway
    (3, 8, 8, 1, 128, 0, 700),         # 72 rows, splits
    (2, 15, 16, 2, 64, 500, 1500),     # 128 rows
    (2, 0, 128, 1, 64, 3, 60),         # one position of 128 heads
    (3, 100, 8, 1, 128, 0, 60),        # windows of several query tiles
])
def test_attention(molt_lib, B, k, Hq, Hkv, D, lo, hi, kn, vn):
    print(f"case B={B} k={k} Hq={Hq} Hkv={Hkv} D={D} ctx=[{lo},{hi}] shift={kn},{vn}", flush=True)
    w = workloads.LAYER_BF16.scaled(batch=B, k=k, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, ctx_lo=lo, ctx_hi=hi)
    layout = workloads.make_kv_layout(w, 23)
    kc, vc = (dev(c) for c in workloads.make_kv_cache(w, layout, 23, 0))
    q = dev(torch.randn(B * (k + 1), Hq, D, generator=workloads.rng(23, "q")).bfloat16())
    args = (dev(torch.from_numpy(layout.block_tables)), dev(torch.from_numpy(layout.context_lens)), k)
    a = molt_lib.paged_attention(q, kc, vc, *args)
    b = molt_lib.paged_attention(q, _shifted(kc, kn), _shifted(vc, vn), *args)
    assert torch.equal(a, b)


@pytest.mark.parametrize("shift", [1, 4])
def test_expert_rows(molt_lib, shift):
    E, rows, d, F = 128, 256, 192, 448
    T = E * rows
    assert moe_plan(BF16, T, 1, E, d, F).big
    g = torch.Generator(device="cuda").manual_seed(shift)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    x, wr, wgu, wd = r(T, d), r(E, d), r(E, 2 * F, d) / 14, r(E, d, F) / 21
    ids = (torch.randperm(T, generator=g, device="cuda") % E).int().view(T, 1)
    a = molt_lib.moe_layer(x, wr, wgu, wd, 1, replay_ids=ids)
    b = molt_lib.moe_layer(_shifted(x, shift), wr, wgu, wd, 1, replay_ids=ids)
    assert torch.equal(a, b)
