"""Launches of three rounds and more in which crowded and nearly empty experts (at most 64 rows) sit side by side deal the two kinds
of tiles to the XCDs by themselves: bit for bit what one workgroup per tile in plain order gives (the other suites check that
against the oracle), for shares on both sides of the lines where the rule starts, the light experts in front, behind and between, 64
experts and fewer, empty ones among them."""
import numpy as np
import pytest
import torch

from paper_2501_16103_amd import binding as mb
from paper_2501_16103_amd import workloads as wk
from tests import helpers as H
from tests.test_gpu_parity import _ids_from_counts

pytestmark = pytest.mark.gpu

MIXES = {
    "worst": [1] * 9 + [700] + [64] * 8 + [600, 0, 513] + [1] * 8 + [900],
    "light first": [3, 64, 0, 17, 1, 33] + [520, 700],
    "light last": [545, 700, 300] + [2, 64, 1],
    "64 experts": ([1] * 7 + [400]) * 8,
    "an eighth": [256] * 7 + [257 + 32, 1, 0],
    "just below": [2048, 1, 2],
}


@pytest.mark.parametrize("dtype,tile_m,tile_n,slack", [("bf16", 256, 256, 0), ("bf16", 256, 256, 32), ("bf16", 128, 256, 0), ("fp8", 256, 256, 0)])
@pytest.mark.parametrize("mix", list(MIXES))
def test_two_kinds(dtype, tile_m, tile_n, slack, mix):
    dev = torch.device("cuda:0")
    counts = MIXES[mix]
    E, T, K = len(counts), sum(counts), 128 if dtype == "fp8" else 64
    ids = _ids_from_counts(counts, 11).to(dev)
    m_tiles = sum(max(1, -(-(c - slack) // tile_m)) for c in counts if c)
    for nt in (-(-768 // m_tiles) - 1, -(-768 // m_tiles), -(-801 // m_tiles)):   # below three rounds, at the line, above it
        N, xs, ws = nt * tile_n, None, None
        wl = wk.Workload("two_kinds", T, E, 1, K, N, *(["fp8"] if dtype == "fp8" else []))
        X, W = wk.make_x(wl, dev), wk.make_w(wl, dev)
        if dtype == "fp8":
            (X, xs), (W, ws) = X, W
        tmap = mb.alloc_task_map(T, 1, E, tile_m, tile_n, N)
        mb.moe_build_task_map_ex(ids, T, 1, E, N, mb.Tiling(tile_m, tile_n, tile_m_slack=slack), tmap)
        out = []
        for mode in (mb.MOE_LAUNCH_PER_TILE, mb.MOE_LAUNCH_AUTO):
            Y = torch.full((T, N), float("nan"), dtype=torch.bfloat16, device=dev)
            mb.moe_grouped_gemm(X, W, None, tmap, Y, mb.GemmDesc(
                mb.MOE_DTYPE_FP8_E4M3 if dtype == "fp8" else mb.MOE_DTYPE_BF16, T, 1, E, K, N, tile_m, tile_n, xs, ws, tile_m_slack=slack,
                launch_mode=mode))
            torch.cuda.synchronize()
            out.append(H.y_bits(Y))
        assert not np.any((out[0] & 0x7FFF) > 0x7F80), "an output was never written"
        assert np.array_equal(out[0], out[1]), f"nt={nt}: {m_tiles * nt} tiles"
