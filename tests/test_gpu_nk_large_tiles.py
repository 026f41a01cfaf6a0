"""[E][N][K] weights on the 256- and 128-row tiles (alternating roles, weight offsets folded into the scalar base, staged
epilogue): row counts around every block edge, one to five k-tiles, several n-tiles."""
import numpy as np
import pytest
import torch

from paper_2501_16103_amd import binding as mb
from paper_2501_16103_amd import workloads as wk
from tests import helpers as H
from tests.test_gpu_neighbours import POISON, _check_swiglu
from tests.test_gpu_parity import _check_y, _ids_from_counts

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    mb.lib()
    return torch.device("cuda:0")


CASES = [
    # tile_m, per-expert row counts (k = 1), K (k-tiles of 64), N
    (256, [256, 1, 64, 65, 128, 0, 129, 145, 160, 161], 64, 256),
    (256, [192, 193, 224, 225, 240, 241, 255, 257, 300], 128, 512),
    (256, [130, 250, 513, 7], 320, 512),
    (128, [128, 1, 63, 64, 65, 0, 127, 129, 193], 64, 256),
    (128, [100, 128, 300], 320, 512),
]


@pytest.mark.parametrize("swiglu", [False, True], ids=["plain", "swiglu"])
@pytest.mark.parametrize("tile_m,counts,K,N", CASES)
def test_nk_large_tiles(dev, oracle_mod, tile_m, counts, K, N, swiglu):
    E, T = len(counts), sum(counts)
    wl = wk.Workload("parity_nk_large", T, E, 1, K, N, "bf16", "gauss_topk", tile_m, 256)
    ids = _ids_from_counts(counts, 11 + E + K)
    X, W = wk.make_x(wl), wk.make_w(wl) * (4.0 if swiglu else 1.0)
    NO, pad = (N // 2 if swiglu else N), 4
    buf = torch.full((T + 2 * pad, NO), POISON, dtype=torch.int16, device=dev)
    tiling = mb.Tiling(tile_m, 256)
    tmap = mb.alloc_task_map(T, 1, E, tile_m, 256, N)
    mb.moe_build_task_map_ex(ids.to(dev), T, 1, E, N, tiling, tmap)
    desc = mb.GemmDesc(mb.MOE_DTYPE_BF16, T, 1, E, K, N, tile_m, 256, w_layout=mb.MOE_W_LAYOUT_NK,
                       epilogue=mb.MOE_EPILOGUE_SWIGLU if swiglu else mb.MOE_EPILOGUE_NONE)
    mb.moe_grouped_gemm(X.to(dev), W.transpose(1, 2).contiguous().to(dev), None, tmap, buf[pad: pad + T], desc)
    torch.cuda.synchronize()
    bits = buf.cpu().numpy().view(np.uint16)
    assert np.all(bits[:pad] == POISON) and np.all(bits[pad + T:] == POISON), "wrote outside Y"
    res = oracle_mod.grouped_gemm_bf16(wk.bits(X), wk.bits(W), ids.numpy())
    Xf, Wf = X.double().numpy(), W.double().numpy()
    if swiglu:
        _check_swiglu(oracle_mod, bits[pad: pad + T], res, Xf, Wf, ids.numpy(), 1, K)
    else:
        _check_y(bits[pad: pad + T], res, Xf, Wf, ids.numpy(), 1, K, H.tol_bf16(K))
