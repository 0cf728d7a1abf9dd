"""Expert GEMMs of bf16 experts with 120 rows on average and more, few of them (too few tiles for the
big-tile kernel: they run on 128-row weight-streaming tiles), at the edges of the tiles: every split
of an expert's rows into 32-row blocks and tiles (0, 1, 33 .. 513 rows), fewer K slices than
the pipeline is deep and counts that no depth divides, last column tiles that are part empty.
The reference takes the SwiGLU product in bf16 as the library stores it; a rounding of it that
goes the other way moves an output by 2^-8 of one of its F terms."""
import pytest
import torch

pytestmark = pytest.mark.gpu

COUNTS = (0, 1, 33, 64, 97, 129, 160, 224, 256, 257, 300, 513)


@pytest.mark.parametrize("d,F", [(64, 64), (128, 192), (192, 320), (320, 128), (576, 448)])
def test_grouped(molt_lib, d, F):
    print(f"case d={d} F={F}", flush=True)
    E, T = len(COUNTS), sum(COUNTS)
    assert T >= 120 * E
    g = torch.Generator(device="cuda").manual_seed(d + F)
    ids = torch.cat([torch.full((c,), e) for e, c in enumerate(COUNTS)]).cuda()
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
