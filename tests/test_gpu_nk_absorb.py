"""[E][N][K] weights on 256 x 256 tiles: an expert's last tile of at most 32 rows is run by the workgroup of the tile before it, where
that saves a round.  Bit for bit what one workgroup per tile of the map gives (the other suites check that against the oracle), with
rests on both sides of 32, none, empty and one-tile experts, one k-tile and more than the weight ring's eleven quarters take to come
round, launches below, at and beyond the sizes where the rule holds, and an order by kind."""
import numpy as np
import pytest
import torch

from paper_2501_16103_amd import binding as mb
from paper_2501_16103_amd import workloads as wk
from tests import helpers as H
from tests.test_gpu_parity import _ids_from_counts

pytestmark = pytest.mark.gpu

COUNTS = [257, 288, 289, 0, 512, 513, 544, 545, 1, 256, 300, 785, 32]


def _absorbs(counts, nt, order):
    """The rule, written down from its description: no more than eight rounds of tiles left, and a round less than the map's own tiles
    fill, where those of at most 128 rows count half and the last round half."""
    total = sum(-(-c // 256) for c in counts) * nt
    left = sum(max(1, -(-(c - 32) // 256)) for c in counts if c) * nt
    few = sum(1 for c in counts if c and (c - 1) % 256 < 128) * nt
    after = -(-left // 256)
    return order != 2 and 256 < total and left <= 2048 and after < -(-total // 256) and after < (total - few / 2) / 256 + 0.5


@pytest.mark.parametrize("K,nt,order,swiglu,absorbs", [
    (64, 9, 0, False, False), (64, 12, 0, True, True), (64, 13, 0, False, False), (128, 22, 0, False, True), (192, 36, 1, False, True),
    (64 * 12, 12, 0, False, True), (64 * 25, 12, 1, True, True), (64 * 25, 24, 0, False, True), (320, 22, 2, False, False),
    (64, 97, 0, True, True), (64, 98, 0, False, False)])
def test_small_last_tiles(K, nt, order, swiglu, absorbs):
    assert _absorbs(COUNTS, nt, order) == absorbs
    dev = torch.device("cuda:0")
    E, T, N = len(COUNTS), sum(COUNTS), nt * 256
    ids = _ids_from_counts(COUNTS, 17).to(dev)
    wl = wk.Workload("nk_absorb", T, E, 1, K, N)
    X, W = wk.make_x(wl, dev), wk.make_w(wl, dev).transpose(1, 2).contiguous()
    tmap = mb.alloc_task_map(T, 1, E, 256, 256, N)
    mb.moe_build_task_map_ex(ids, T, 1, E, N, mb.Tiling(256, 256, order), tmap)
    out = []
    for mode in (mb.MOE_LAUNCH_PER_TILE, mb.MOE_LAUNCH_AUTO):
        Y = torch.full((T, N // 2 if swiglu else N), float("nan"), dtype=torch.bfloat16, device=dev)
        mb.moe_grouped_gemm(X, W, None, tmap, Y, mb.GemmDesc(
            mb.MOE_DTYPE_BF16, T, 1, E, K, N, 256, 256, w_layout=mb.MOE_W_LAYOUT_NK, launch_mode=mode,
            epilogue=mb.MOE_EPILOGUE_SWIGLU if swiglu else mb.MOE_EPILOGUE_NONE))
        torch.cuda.synchronize()
        out.append(H.y_bits(Y))
    assert not np.any((out[0] & 0x7FFF) > 0x7F80), "an output was never written"
    assert np.array_equal(out[0], out[1])
