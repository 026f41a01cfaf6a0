"""Which form of launch a product on 16-row tiles takes (host only)."""
import pytest

from paper_2501_16103_amd import binding as mb

BF16, FP8 = mb.MOE_DTYPE_BF16, mb.MOE_DTYPE_FP8_E4M3
THREADS = {  # threads of a workgroup, by tile width: the forms of one workgroup per tile
    mb.MOE_ROWS16_PER_TILE_DEEP: {256: 512, 128: 256},
    mb.MOE_ROWS16_PER_TILE: {256: 512, 128: 256},
    mb.MOE_ROWS16_PER_TILE_SMALL: {256: 128, 128: 128},
}


def _grid(T, k, E, tile_n, N):
    return (mb.moe_grid_upper_bound(T, k, E, 16, tile_n, N) + 7) // 8 * 8 + 16


@pytest.mark.parametrize("dtype", [BF16, FP8])
@pytest.mark.parametrize("tile_n,E,K,N,T", [
    (256, 256, 1, 2048, 65536),     # 2^23 + 2048 tiles, streaming refused: one k-tile
    (256, 512, 1, 2048, 32768),     # ... and more than 256 experts
    (128, 256, 1, 2048, 65536),     # 2^24 + 4096 narrow ones
    (128, 512, 2, 2048, 32768),
    (128, 256, 3, 32768, 4096),     # K below every ring
])
def test_a_launch_of_too_many_work_items_takes_two_wavefronts(dtype, tile_n, E, K, N, T):
    K *= 64 if dtype == BF16 else 128
    form = mb.moe_rows16_launch(dtype, tile_n, T, E, E, K, N, mb.MOE_LAUNCH_PER_TILE)
    assert form == mb.MOE_ROWS16_PER_TILE_SMALL
    assert mb.moe_rows16_launch(dtype, tile_n, T, E, E, K, N) in (form, mb.MOE_ROWS16_STREAM_SHORT_K, mb.MOE_ROWS16_PAIRS_MERGED, mb.MOE_ROWS16_PAIRS)
    if K == (64 if dtype == BF16 else 128):
        assert mb.moe_rows16_launch(dtype, tile_n, T, E, E, K, N) == form


@pytest.mark.parametrize("dtype", [BF16, FP8])
@pytest.mark.parametrize("mode", [mb.MOE_LAUNCH_AUTO, mb.MOE_LAUNCH_PER_TILE, mb.MOE_LAUNCH_RESIDENT])
@pytest.mark.parametrize("tile_n", [256, 128])
def test_no_form_of_one_workgroup_per_tile_overflows(dtype, mode, tile_n):
    """Up to the most rows a map holds and beyond the widest product: every launch fits 2^32 - 1 work items or is refused."""
    bk, seen, refused = 64 if dtype == BF16 else 128, set(), 0
    for E in (1, 8, 255, 256, 257, 512, 1024):
        for k in (1, E):
            for k_tiles in (1, 2, 3, 4, 5, 6, 40):
                for T in (1, 77, (1 << 20) // k, (1 << 24) // k):
                    for N in (256, 2048, 4096 + 256, 32768, 65536, 1 << 20):
                        if T < 1:
                            continue
                        form = mb.moe_rows16_launch(dtype, tile_n, T, k, E, k_tiles * bk, N, mode)
                        grid = _grid(T, k, E, tile_n, N)
                        seen.add(form)
                        if form == mb.MOE_ERR_UNSUPPORTED:
                            refused += 1
                            assert grid * 128 >= 1 << 32
                        elif form in THREADS:
                            assert grid * THREADS[form][tile_n] < 1 << 32, (E, k, k_tiles, T, N)
                            if form == mb.MOE_ROWS16_PER_TILE_SMALL:
                                assert grid * THREADS[mb.MOE_ROWS16_PER_TILE][tile_n] >= 1 << 32
    assert mb.MOE_ROWS16_PER_TILE_SMALL in seen and mb.MOE_ROWS16_PER_TILE in seen and refused


@pytest.mark.parametrize("args,want", [
    ((BF16, 256, 1, 1, 8, 64, 512, -1), mb.MOE_ERR_INVALID_ARG),
    ((2, 256, 1, 1, 8, 64, 512, 0), mb.MOE_ERR_INVALID_ARG),
    ((BF16, 256, 1, 9, 8, 64, 512, 0), mb.MOE_ERR_INVALID_ARG),
    ((BF16, 64, 1, 1, 8, 64, 512, 0), mb.MOE_ERR_UNSUPPORTED),
    ((BF16, 256, 1, 1, 8, 96, 512, 0), mb.MOE_ERR_UNSUPPORTED),
    ((FP8, 128, 1, 1, 8, 64, 512, 0), mb.MOE_ERR_UNSUPPORTED),
    ((BF16, 256, 1, 1, 8, 64, 384, 0), mb.MOE_ERR_UNSUPPORTED),
    ((BF16, 256, 1, 1, 2000, 64, 512, 0), mb.MOE_ERR_UNSUPPORTED),
])
def test_form_of_what_the_product_refuses(args, want):
    assert mb.moe_rows16_launch(*args) == want


@pytest.mark.parametrize("dtype,tile_n,E,k,K,N,T,want", [
    (FP8, 128, 64, 6, 512, 1408, 100, mb.MOE_ROWS16_PER_TILE),            # 1111 tiles at most: two per workgroup of a streaming launch
    (FP8, 128, 256, 8, 512, 3968, 128, mb.MOE_ROWS16_STREAM_SHORT_K),     # sixteen tiles per CU, 4 rows per expert
    (FP8, 128, 256, 8, 512, 3968, 383, mb.MOE_ROWS16_STREAM_SHORT_K),
    (FP8, 128, 256, 8, 512, 3968, 384, mb.MOE_ROWS16_PER_TILE),           # ... 12
    (FP8, 128, 256, 8, 512, 2176, 45, mb.MOE_ROWS16_PER_TILE),            # 3303 tiles expected
    (FP8, 128, 256, 8, 384, 3968, 128, mb.MOE_ROWS16_PER_TILE),           # three k-tiles: below this ring too
    (FP8, 256, 256, 8, 256, 2816, 64, mb.MOE_ROWS16_PER_TILE),
    (BF16, 256, 256, 8, 128, 2048, 64, mb.MOE_ROWS16_STREAM_SHORT_K),     # no scales: from two tiles per workgroup on
    (BF16, 128, 128, 8, 320, 1408, 64, mb.MOE_ROWS16_STREAM_SHORT_K),
    (BF16, 256, 64, 6, 128, 1024, 64, mb.MOE_ROWS16_PER_TILE_DEEP),
])
def test_short_k_streams_where_two_workgroups_fit_a_cu_and_lead(dtype, tile_n, E, k, K, N, T, want):
    assert mb.moe_rows16_launch(dtype, tile_n, T, k, E, K, N) == want
    if K // (64 if dtype == BF16 else 128) >= (2 if tile_n == 256 else 4):
        assert mb.moe_rows16_launch(dtype, tile_n, T, k, E, K, N, mb.MOE_LAUNCH_RESIDENT) == mb.MOE_ROWS16_STREAM_SHORT_K


@pytest.mark.parametrize("T,k,E,K,N,tile_n,want", [
    (64, 1, 64, 192, 2816, 256, 1),
    (65, 1, 64, 192, 2816, 256, 2),     # more rows than a wavefront has lanes
    (16, 4, 65, 192, 2816, 256, 2),     # ... experts
    (64, 1, 64, 128, 2816, 256, 2),     # a K shorter than the ring
    (32, 2, 4, 1024, 32768, 256, 2),    # an expert's rows run as one tile
    (32, 2, 4, 1024, 32768, 128, 2),
    (8, 8, 64, 192, 5 * 128, 128, 1),
    (64, 1, 64, 192, 11 * 128, 128, 2),     # more than one narrow tile per CU, and no pairs
])
def test_one_launch_for_maps_and_product(T, k, E, K, N, tile_n, want):
    d = dict(dtype=BF16, T=T, k=k, E=E, K=K, N=N, tile_m=16, tile_n=tile_n)
    g = mb.Tiling(16, tile_n)
    assert mb.moe_pair_gemm_launches(T, k, E, N, g, mb.GemmDesc(**d)) == want
    for other in (dict(dtype=FP8, K=K * 2), dict(w_layout=mb.MOE_W_LAYOUT_NK), dict(launch_mode=1), dict(launch_mode=2), dict(T=T + 1), dict(tile_m=32),
                  dict(tile_m_slack=4), dict(tile_m_small=16), dict(K=K + 32), dict(epilogue=7)):
        assert mb.moe_pair_gemm_launches(T, k, E, N, g, mb.GemmDesc(**{**d, **other})) == 2
    for tiling in (mb.Tiling(16, tile_n, order=1), mb.Tiling(32, tile_n), mb.Tiling(128, tile_n, tile_m_small=16, small_max_rows=8)):
        assert mb.moe_pair_gemm_launches(T, k, E, N, tiling, mb.GemmDesc(**d)) == 2
