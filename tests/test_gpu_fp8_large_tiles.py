"""fp8 tiles of 64 rows and more: the 256-row loop in alternating roles with one k-step per k-tile, and the narrower
functions on 32-row blocks, at row counts around every block and tile edge and at one to five k-tiles."""
import pytest
import torch

from paper_2501_16103_amd import binding as mb
from paper_2501_16103_amd import workloads as wk
from tests import helpers as H
from tests.test_gpu_neighbours import _check_swiglu, _run_swiglu
from tests.test_gpu_parity import _check_y, _ids_from_counts, _run_gemm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    mb.lib()
    return torch.device("cuda:0")


CASES = [
    # tile_m, per-expert row counts (k = 1), K (k-tiles of 128), N
    (256, [256, 1, 33, 64, 65, 97, 128, 0, 129, 145], 128, 256),        # one k-tile
    (256, [160, 161, 192, 193, 224, 225, 240, 241, 255], 256, 256),     # every count of live 16-row blocks, two k-tiles
    (256, [257, 300, 384, 513, 600], 384, 512),                         # several m-tiles, three k-tiles
    (256, [130, 250, 256, 7], 640, 256),                                # five: three steady iterations, two that fetch nothing
    (64, [1, 31, 32, 33, 63, 64, 65, 128, 130], 128, 256),
    (64, [64, 200, 17], 512, 512),
]


@pytest.mark.parametrize("swiglu", [False, True], ids=["plain", "swiglu"])
@pytest.mark.parametrize("tile_m,counts,K,N", CASES)
def test_fp8_large_tiles(dev, oracle_mod, tile_m, counts, K, N, swiglu):
    E, T = len(counts), sum(counts)
    wl = wk.Workload("parity_fp8_large", T, E, 1, K, N, "fp8", "gauss_topk", tile_m, 256)
    ids = _ids_from_counts(counts, 3 + E + K)
    X, xs = wk.make_x(wl)
    W, ws = wk.make_w(wl)
    if swiglu:
        ws = ws * 4.0
    got = (_run_swiglu if swiglu else _run_gemm)(dev, wl, ids, X, W, xs, ws)
    res = oracle_mod.grouped_gemm_fp8(wk.bits(X), wk.bits(W), xs.numpy(), ws.numpy(), ids.numpy())
    Xf = X.view(torch.float8_e4m3fn).double().numpy()
    Wf = W.view(torch.float8_e4m3fn).double().numpy()
    sx, sw = xs.double().numpy(), ws.double().numpy()
    if swiglu:
        _check_swiglu(oracle_mod, got, res, Xf, Wf, ids.numpy(), 1, K, sx, sw)
    else:
        _check_y(got, res, Xf, Wf, ids.numpy(), 1, K, H.tol_fp8(K), sx, sw)
