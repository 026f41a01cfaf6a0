"""Tilings that a layer plan takes other than the library's default (host only)."""
import pytest

from paper_2501_16103_amd import binding as mb


@pytest.mark.parametrize("T,k,E,hidden,inter,want", [
    (32, 2, 8, 4096, 14336, (16, 256)),     # 8 rows per expert: the default
    (33, 2, 8, 4096, 14336, (16, 256)),     # 9 to 32 rows, 896 wide tiles: streamed
    (128, 2, 8, 4096, 14336, (16, 256)),
    (129, 2, 8, 4096, 14336, (256, 256)),
    (64, 2, 8, 4096, 7168, (16, 256)),      # 448 wide tiles
    (64, 2, 8, 4096, 7040, (256, 256)),     # 440, N a multiple of 256 only
    (64, 2, 8, 4096, 6656, (16, 256)),      # 416
    (64, 2, 8, 4096, 6144, (16, 256)),      # 384
    (64, 2, 8, 4096, 5888, (256, 256)),     # 368
    (64, 2, 8, 3840, 14336, (16, 256)),     # any K from which the streamed tiles are merged on
    (64, 2, 8, 1024, 14336, (16, 256)),
    (64, 2, 8, 768, 14336, (256, 256)),
    (64, 4, 16, 4096, 8192, (16, 256)),     # 1024 wide tiles, 16 experts
    (128, 4, 16, 4096, 8192, (16, 256)),
    (64, 4, 17, 4096, 8192, (16, 256)),     # 1088
    (128, 4, 32, 2048, 8192, (16, 256)),    # 2048
    (128, 4, 32, 2048, 8448, (256, 256)),   # 2112
    (128, 4, 36, 4096, 4096, (256, 256)),   # 1152, more than 32 experts
    (102, 4, 24, 4096, 4096, (256, 256)),   # 17 rows per expert, more than 16 experts
    (96, 4, 24, 4096, 4096, (16, 256)),     # 16
    (36, 2, 8, 4096, 7168, (16, 256)),      # 9 rows: merging the 448 tiles would not save a round, but the second one has room
    (36, 2, 8, 4096, 6656, (16, 256)),
    (36, 2, 8, 4096, 6144, (256, 256)),     # ... 384
    (54, 2, 12, 2048, 5120, (256, 256)),    # ... 480: little room
    (76, 4, 32, 2048, 1792, (256, 256)),    # ... 448, more experts
    (36, 2, 8, 768, 7168, (256, 256)),
    (64, 2, 8, 2048, 11008, (16, 256)),     # N a multiple of 512: up to 48 experts and 16 rows
    (65, 2, 8, 2048, 11008, (256, 256)),
    (128, 6, 48, 2048, 1792, (16, 256)),
    (152, 6, 64, 2048, 1280, (256, 256)),
    (152, 6, 64, 2048, 1536, (16, 256)),    # ... of 1024
    (152, 6, 64, 2048, 1408, (256, 256)),
    (256, 8, 128, 2048, 1024, (16, 256)),
    (400, 8, 256, 4096, 512, (16, 256)),
    (65, 4, 16, 2048, 4096, (256, 256)),    # 17 rows, 512 tiles: no room in the last round
    (64, 4, 16, 2048, 4096, (16, 256)),
    (65, 4, 16, 2048, 3584, (16, 256)),     # ... 448
    (400, 8, 257, 4096, 256, (256, 256)),   # more experts than a launch streams
    (400, 8, 300, 4096, 256, (256, 256)),
    (600, 8, 384, 4096, 256, (256, 256)),
    (768, 8, 512, 4096, 256, (256, 256)),
    (777, 6, 64, 2048, 1408, (128, 256)),
])
def test_tiling_of_the_first_product(T, k, E, hidden, inter, want):
    plan = mb.MoeLayerPlan(T, k, E, hidden, inter, "cpu")
    assert (plan.g1.tile_m, plan.g1.tile_n) == want
    assert (plan.d1.tile_m, plan.d1.tile_n, plan.d1.tile_m_slack) == (plan.g1.tile_m, plan.g1.tile_n, plan.g1.tile_m_slack)
    assert mb.moe_tiling_supported(mb.MOE_DTYPE_BF16, plan.g1)
