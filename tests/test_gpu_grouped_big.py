"""The grouped big-tile expert GEMMs (bf16) where the plan takes them, at the edges of their tiles: every
split of an expert's rows into 32-row blocks, halves and tiles (0, 1, 33 .. 513 rows: halves of different
heights, an empty second half, several tiles), over enough experts to fill the chip; one K slice and
counts that no depth divides, last column tiles that are part empty. The reference takes the SwiGLU
product in bf16 as the library stores it; a rounding of it that goes the other way moves an output by
2^-8 of one of its F terms."""
import pytest
import torch

from plans import BF16, moe_plan

pytestmark = pytest.mark.gpu

COUNTS = (0, 1, 33, 64, 97, 129, 160, 224, 256, 257, 300, 513)


@pytest.mark.parametrize("d,F,repeat", [(64, 320, 13), (128, 128, 11), (192, 320, 12), (320, 192, 9), (576, 64, 13),
                                        (448, 448, 7), (1088, 1088, 2)])
def test_grouped(molt_lib, d, F, repeat):
    print(f"case d={d} F={F} repeat={repeat}", flush=True)
    counts = COUNTS * repeat
    E, T = len(counts), sum(counts)
    assert moe_plan(BF16, T, 1, E, d, F).big
    g = torch.Generator(device="cuda").manual_seed(d + F)
    ids = torch.cat([torch.full((c,), e) for e, c in enumerate(counts)]).cuda()
    ids = ids[torch.randperm(T, generator=g, device="cuda")].int().view(T, 1)
    x = torch.randn(T, d, generator=g, device="cuda").bfloat16()
    wr = torch.randn(E, d, generator=g, device="cuda").bfloat16()
    wgu = (torch.randn(E, 2 * F, d, generator=g, device="cuda") / d ** 0.5).bfloat16()
    wd = (torch.randn(E, d, F, generator=g, device="cuda") / F ** 0.5).bfloat16()
    out = molt_lib.moe_layer(x, wr, wgu, wd, 1, replay_ids=ids)     # K = 1: weight 1
    again = molt_lib.moe_layer(x, wr, wgu, wd, 1, replay_ids=ids)
    ref = torch.zeros(T, d, dtype=torch.float64, device="cuda")
    lim = torch.zeros(T, d, dtype=torch.float64, device="cuda")
    for e in range(E):
        t = (ids[:, 0] == e).nonzero()[:, 0]
        v = x[t].double() @ wgu[e].double().T
        h = (v[:, :F] * torch.sigmoid(v[:, :F]) * v[:, F:]).bfloat16().double()
        ref[t] = h @ wd[e].double().T
        # f32 sums, and one bf16 step in the few products near a rounding boundary
        lim[t] = 2.0 ** -20 * (h.abs() @ wd[e].double().abs().T) + \
            4 * 2.0 ** -8 * h.abs().amax(1, keepdim=True) * wd[e].double().abs().amax(1)
    assert bool(((out.double() - ref).abs() <= lim).all())
    assert torch.equal(out, again)
