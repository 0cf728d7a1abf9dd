"""The choice between the grouped expert GEMM kernels, on the host: big tiles where they fill the chip,
the weight-streaming kernel for few experts, few rows, and operands past 32-bit offsets."""
import pytest

from plans import BF16, F32, FP8, moe_plan


@pytest.mark.parametrize("T,K,E,d,F", [(4000, 8, 128, 2048, 768), (2304, 8, 128, 2048, 768), (4096, 8, 64, 2048, 1408),
                                       (8192, 2, 8, 2048, 768), (4000, 1, 1, 2048, 6144), (2048, 2, 8, 4096, 14336)])
def test_big_tiles_fill_the_chip(T, K, E, d, F):
    p = moe_plan(BF16, T, K, E, d, F)
    assert p.big and p.tile_m == 256


@pytest.mark.parametrize("T,K,E,d,F", [
    (512, 2, 8, 2048, 768), (1024, 2, 8, 2048, 768),      # 128 and 256 rows of few experts
    (256, 1, 1, 2048, 6144), (1024, 1, 1, 2048, 768), (1024, 1, 1, 4096, 1408),   # one expert
    (512, 2, 4, 2048, 768), (1024, 1, 4, 1024, 2048), (4096, 1, 16, 512, 256),
])
def test_few_tiles_stay_on_the_streaming_kernel(T, K, E, d, F):
    p = moe_plan(BF16, T, K, E, d, F)
    assert not p.big and p.tile_m == 128


def test_types_rows_and_offsets():
    assert (moe_plan(F32, 4000, 8, 128, 2048, 768).tile_m, moe_plan(F32, 4000, 8, 128, 2048, 768).big) == (32, False)
    assert not moe_plan(FP8, 4000, 8, 128, 2048, 768).big
    for T, tile in ((384, 32), (385, 64), (896, 64), (897, 128), (1900, 128)):
        p = moe_plan(BF16, T, 8, 128, 2048, 768)
        assert (p.tile_m, p.big) == (tile, False), T
    assert moe_plan(BF16, 32767, 8, 128, 2048, 768).big and not moe_plan(BF16, 32768, 8, 128, 2048, 768).big
