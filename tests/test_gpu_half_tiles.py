"""Launches whose last round of tiles is short run those tiles as two half tiles each: bit for bit what one workgroup per
tile gives (the other suites check that against the oracle), for rests from none to more than half a round (1 and 16 tiles of
an XCD's 32 behind a full round among them, which the test asserts from the map), with and without full rounds in front, row counts of every task function, slack rows, the fused activation and both block orders."""
import numpy as np
import pytest
import torch

from paper_2501_16103_amd import binding as mb
from paper_2501_16103_amd import workloads as wk
from tests import helpers as H
from tests.test_gpu_parity import _ids_from_counts

pytestmark = pytest.mark.gpu

COUNTS = {256: [256, 288, 1, 64, 65, 128, 129, 0, 200, 260, 513, 17, 270], 128: [128, 1, 64, 65, 129, 100, 0, 33, 300]}


def _tiles_of_xcd(header, xcd):
    """Tiles that XCD `xcd` of 8 runs: a contiguous share of all, or of the heavy and of the light ones (order 2)."""
    total = int(header[mb.HDR["TOTAL_TILES"]])
    if int(header[mb.HDR["SIGMA_ORDER"]]) == 2:
        heavy = int(header[mb.HDR["HEAVY_TILES"]])
        return sum(n * (xcd + 1) // 8 - n * xcd // 8 for n in (heavy, total - heavy))
    share = -(-total // 8)
    return max(0, min(share, total - xcd * share))


@pytest.mark.parametrize("dtype,tile_m,tile_n,slack", [("bf16", 256, 256, 0), ("bf16", 256, 256, 32), ("bf16", 128, 256, 0),
                                                       ("bf16", 128, 128, 0), ("fp8", 256, 256, 0)])
def test_half_tiles(dtype, tile_m, tile_n, slack):
    dev = torch.device("cuda:0")
    counts = COUNTS[tile_m]
    E, T = len(counts), sum(counts)
    ids = _ids_from_counts(counts, 9).to(dev)
    seen = set()   # (full rounds in front, tiles in the last round) of every XCD
    for K, nt, order, swiglu in ((64, 1, 0, False), (192, 1, 0, True), (64, 8, 0, False), (128, 9, 0, True), (128, 13, 0, False),
                                 (64, 17, 2, False), (320, 19, 0, False), (64, 23, 1, True), (64, 31, 0, False),
                                 (64, 18, 0, False), (64, 20, 0, True), (64, 24, 0, False), (64, 29, 0, False), (64, 34, 2, False), (64, 40, 0, False)):
        N, xs, ws = nt * tile_n, None, None
        if dtype == "fp8":
            K *= 2
            wl = wk.Workload("half_tiles", T, E, 1, K, N, "fp8")
            (X, xs), (W, ws) = wk.make_x(wl, dev), wk.make_w(wl, dev)
        else:
            wl = wk.Workload("half_tiles", T, E, 1, K, N)
            X, W = wk.make_x(wl, dev), wk.make_w(wl, dev)
        tmap = mb.alloc_task_map(T, 1, E, tile_m, tile_n, N)
        mb.moe_build_task_map_ex(ids, T, 1, E, N, mb.Tiling(tile_m, tile_n, order, 0, 0, slack), tmap)
        out = []
        for mode in (mb.MOE_LAUNCH_PER_TILE, mb.MOE_LAUNCH_AUTO):
            Y = torch.full((T, N // 2 if swiglu else N), float("nan"), dtype=torch.bfloat16, device=dev)
            mb.moe_grouped_gemm(X, W, None, tmap, Y, mb.GemmDesc(
                mb.MOE_DTYPE_FP8_E4M3 if dtype == "fp8" else mb.MOE_DTYPE_BF16, T, 1, E, K, N, tile_m, tile_n, xs, ws, tile_m_slack=slack, launch_mode=mode,
                epilogue=mb.MOE_EPILOGUE_SWIGLU if swiglu else mb.MOE_EPILOGUE_NONE))
            torch.cuda.synchronize()
            out.append(H.y_bits(Y))
        header = tmap[:32].cpu()
        total = int(header[mb.HDR["TOTAL_TILES"]])
        seen |= {divmod(_tiles_of_xcd(header, x), 32) for x in range(8)}
        assert not np.any((out[0] & 0x7FFF) > 0x7F80), "an output was never written"
        assert np.array_equal(out[0], out[1]), f"K={K} nt={nt} order={order}: {total} tiles, {-(-total // 8) % 32} left over"
    rests = {(full > 0, rest) for full, rest in seen}
    assert (True, 1) in rests and (True, 16) in rests, "halved rests at both ends behind a full round"
    assert any(not full and 1 <= rest <= 16 for full, rest in rests), "a launch of halves only"
    assert any(full and rest > 16 for full, rest in rests) and any(not full and rest > 16 for full, rest in rests), "rests that stay whole"
