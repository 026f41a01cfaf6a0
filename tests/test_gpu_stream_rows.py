"""16-row tiles streamed with up to 64 (128-wide tiles: 32) rows of an expert at a time: bit for bit what one workgroup per 16-row tile
gives (the other suites check that against the oracle), for row counts around every number of blocks in changing order, so that
neighbouring tiles run different copies of the loop, for one to several tiles per workgroup, more than 64 experts, and both sides of the
lines in rows and in K where the rule starts."""
import numpy as np
import pytest
import torch

from paper_2501_16103_amd import binding as mb
from paper_2501_16103_amd import workloads as wk
from tests import helpers as H
from tests.test_gpu_parity import _ids_from_counts

pytestmark = pytest.mark.gpu

MIXED = [1, 64, 16, 65, 17, 0, 32, 33, 15, 48, 3, 129, 2, 31, 63, 1]                 # 33 rows on average: beyond the line
AROUND = [1, 64, 16, 65, 17, 0, 32, 33, 15, 1, 3, 80, 2, 31, 8, 1]                   # 23
THIN = [1, 8, 16, 17, 0, 33, 2, 9]                                                   # 10


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("tile_n,counts,K16,nt,swiglu", [
    (256, AROUND, 16, 5, False), (256, AROUND, 16, 40, True), (128, AROUND, 17, 10, False), (128, AROUND, 16, 21, True), (128, AROUND, 16, 60, False),
    (256, THIN * 10, 16, 9, False), (128, THIN * 10, 16, 11, True), (256, THIN * 25, 16, 3, False), (256, AROUND, 15, 20, False),
    (256, MIXED, 16, 20, False), (128, MIXED, 16, 33, False)])
def test_rows_of_several_tiles(dtype, tile_n, counts, K16, nt, swiglu):
    dev = torch.device("cuda:0")
    E, T, N = len(counts), sum(counts), nt * tile_n
    K = K16 * (128 if dtype == "fp8" else 64)
    ids, xs, ws = _ids_from_counts(counts, 7).to(dev), None, None
    wl = wk.Workload("stream_rows", T, E, 1, K, N, *(["fp8"] if dtype == "fp8" else []))
    X, W = wk.make_x(wl, dev), wk.make_w(wl, dev)
    if dtype == "fp8":
        (X, xs), (W, ws) = X, W
    tmap = mb.alloc_task_map(T, 1, E, 16, tile_n, N)
    mb.moe_build_task_map_ex(ids, T, 1, E, N, mb.Tiling(16, tile_n), tmap)
    out = []
    for mode in (mb.MOE_LAUNCH_PER_TILE, mb.MOE_LAUNCH_AUTO, mb.MOE_LAUNCH_RESIDENT, 8, 24):   # the last two: so many workgroups
        Y = torch.full((T, N // 2 if swiglu else N), float("nan"), dtype=torch.bfloat16, device=dev)
        mb.moe_grouped_gemm(X, W, None, tmap, Y, mb.GemmDesc(
            mb.MOE_DTYPE_FP8_E4M3 if dtype == "fp8" else mb.MOE_DTYPE_BF16, T, 1, E, K, N, 16, tile_n, xs, ws, launch_mode=mode,
            epilogue=mb.MOE_EPILOGUE_SWIGLU if swiglu else mb.MOE_EPILOGUE_NONE))
        torch.cuda.synchronize()
        out.append(H.y_bits(Y))
    assert not np.any((out[0] & 0x7FFF) > 0x7F80), "an output was never written"
    for o in out[1:]:
        assert np.array_equal(out[0], o)
