"""Resident 16-row launches against one workgroup per tile, bit for bit: shares of less than one, one to two and many tiles
per workgroup, 128-wide tiles run in pairs (an even number of n-tiles) and singly (an odd one, or K too short for the pair's
ring).  [E][N][K] weights have one launch, one workgroup per tile, in every mode: those rows are checked against the oracle only."""
import pytest
import torch

from paper_2501_16103_amd import binding as mb
from paper_2501_16103_amd import workloads as wk
from tests import helpers as H
from tests.test_gpu_neighbours import _check_swiglu
from tests.test_gpu_parity import _check_y

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, layout, tile_n, T, E, k, K, N, routing, swiglu, modes
    ("bf16", "kn", 128, 40, 16, 2, 448, 768, "gauss_topk", False, (8, 16, 64, 96, 2)),
    ("bf16", "kn", 128, 40, 16, 2, 448, 640, "gauss_topk", True, (8, 64, 2)),
    ("bf16", "kn", 128, 33, 8, 2, 128, 512, "zipf", False, (8, 2)),          # two k-tiles: no ring is filled
    ("bf16", "kn", 256, 90, 8, 2, 192, 768, "zipf", True, (8, 24, 64, 2)),   # several m-tiles per expert
    ("bf16", "nk", 256, 90, 8, 2, 256, 768, "zipf", False, ()),
    ("fp8", "kn", 128, 32, 64, 6, 384, 512, "uniform_topk", False, (8, 128, 2)),
    ("fp8", "nk", 128, 32, 64, 6, 512, 512, "uniform_topk", True, ()),
    ("fp8", "nk", 256, 50, 16, 2, 896, 512, "zipf", False, ()),
    ("fp8", "kn", 256, 50, 200, 2, 128, 512, "zipf", False, (8, 2)),         # one k-tile, four groups of task records
    # K too short for the deep ring: resident in the form of two workgroups per CU
    ("bf16", "kn", 256, 60, 32, 2, 128, 512, "gauss_topk", True, (8, 32, 2)),
    ("bf16", "kn", 128, 60, 32, 2, 320, 384, "zipf", False, (8, 32, 2)),
    ("fp8", "kn", 256, 60, 32, 2, 256, 512, "zipf", False, (8, 32, 2)),
    ("fp8", "kn", 128, 60, 32, 2, 512, 640, "gauss_topk", True, (8, 32, 2)),
    # ... with the most scales that a streaming launch holds (T + E = 2048)
    ("fp8", "kn", 128, 1984, 64, 1, 512, 384, "zipf", False, (8, 64, 2)),
    # more tiles than CUs, one workgroup per tile, two per CU (more than 256 experts, or T + E > 2048)
    ("bf16", "kn", 256, 100, 300, 4, 192, 512, "gauss_topk", False, (2,)),
    ("bf16", "kn", 128, 100, 300, 4, 384, 256, "zipf", True, (2,)),
    ("fp8", "kn", 256, 100, 300, 4, 128, 512, "zipf", True, (2,)),
    ("fp8", "kn", 128, 2000, 64, 1, 256, 256, "gauss_topk", False, (2,)),
    # the same with 32 k-tiles and more than two 256-wide tiles per CU: the deep form
    ("bf16", "kn", 256, 100, 300, 4, 2048, 768, "gauss_topk", False, (2,)),
]


@pytest.mark.parametrize("dtype,layout,tile_n,T,E,k,K,N,routing,swiglu,modes", CASES)
def test_stream_shares(oracle_mod, dtype, layout, tile_n, T, E, k, K, N, routing, swiglu, modes):
    dev = torch.device("cuda:0")
    wl = wk.Workload("stream_shares", T, E, k, K, N, dtype, routing, 16, tile_n)
    fp8, dt = dtype == "fp8", mb.MOE_DTYPE_FP8_E4M3 if dtype == "fp8" else mb.MOE_DTYPE_BF16
    ids, xs, ws = wk.make_routing(wl), None, None
    if fp8:
        (X, xs), (W, ws) = wk.make_x(wl), wk.make_w(wl)
        ws = ws * (4.0 if swiglu else 1.0)
    else:
        X, W = wk.make_x(wl), wk.make_w(wl) * (4.0 if swiglu else 1.0)
    Wd = (W.transpose(1, 2).contiguous() if layout == "nk" else W).to(dev)
    Xd, xd, wd = X.to(dev), None if xs is None else xs.to(dev), None if ws is None else ws.to(dev)
    tmap = mb.alloc_task_map(T, k, E, 16, tile_n, N)
    mb.moe_build_task_map(ids.to(dev), T, k, E, 16, tile_n, N, tmap)

    def run(mode):
        Y = torch.full((T * k, N // 2 if swiglu else N), float("nan"), dtype=torch.bfloat16, device=dev)
        mb.moe_grouped_gemm(Xd, Wd, None, tmap, Y, mb.GemmDesc(
            dt, T, k, E, K, N, 16, tile_n, xd, wd, epilogue=mb.MOE_EPILOGUE_SWIGLU if swiglu else mb.MOE_EPILOGUE_NONE,
            w_layout=mb.MOE_W_LAYOUT_NK if layout == "nk" else mb.MOE_W_LAYOUT_KN, launch_mode=mode))
        torch.cuda.synchronize()
        return H.y_bits(Y)

    want = run(mb.MOE_LAUNCH_PER_TILE)
    for mode in modes + ((mb.MOE_LAUNCH_AUTO,) if layout == "kn" else ()):
        assert (run(mode) == want).all(), f"launch mode {mode}"
    if fp8:
        res = oracle_mod.grouped_gemm_fp8(wk.bits(X), wk.bits(W), xs.numpy(), ws.numpy(), ids.numpy())
        Xf, Wf = X.view(torch.float8_e4m3fn).double().numpy(), W.view(torch.float8_e4m3fn).double().numpy()
        sc = (xs.double().numpy(), ws.double().numpy())
    else:
        res = oracle_mod.grouped_gemm_bf16(wk.bits(X), wk.bits(W), ids.numpy())
        Xf, Wf, sc = X.double().numpy(), W.double().numpy(), (None, None)
    if swiglu:
        _check_swiglu(oracle_mod, want, res, Xf, Wf, ids.numpy(), k, K, *sc)
    else:
        _check_y(want, res, Xf, Wf, ids.numpy(), k, K, H.tol_fp8(K) if fp8 else H.tol_bf16(K), *sc)


def test_more_tiles_than_work_items_of_the_deep_form():
    """2^23 + 4096 tiles of 256 columns: more than a launch of 512 threads per tile can hold, not more than one of 128."""
    dev, T, E, K, N = torch.device("cuda:0"), 32768, 512, 64, 2048
    g = torch.Generator(device=dev).manual_seed(5)
    X = torch.randn(T, K, generator=g, device=dev).to(torch.bfloat16)
    W = (torch.randn(E, K, N, generator=g, device=dev) / 8).to(torch.bfloat16)
    ids = torch.arange(E, dtype=torch.int32, device=dev).expand(T, E).contiguous()      # every token to every expert
    tmap = mb.alloc_task_map(T, E, E, 16, 256, N)
    mb.moe_build_task_map(ids, T, E, E, 16, 256, N, tmap)
    Y = torch.empty(T, E, N // 2, dtype=torch.bfloat16, device=dev)
    mb.moe_grouped_gemm(X, W, ids, tmap, Y, mb.GemmDesc(mb.MOE_DTYPE_BF16, T, E, E, K, N, 16, 256, epilogue=mb.MOE_EPILOGUE_SWIGLU))
    for e in (0, 1, 255, 256, 510, 511):
        gate, up = (X.double() @ W[e].double()).split(N // 2, dim=1)
        want = (torch.nn.functional.silu(gate) * up).to(torch.bfloat16).double()
        # one bf16 rounding each, and K * 2^-24 of sums of at most about 4 * |x||w| in front of it
        assert ((Y[:, e].double() - want).abs() <= 2.0 ** -7 * want.abs() + 1e-4).all(), f"expert {e}"


@pytest.mark.parametrize("tile_n,K", [(256, 64), (128, 128)])
def test_more_tiles_than_work_items_where_tiles_could_stream(tile_n, K):
    """The same with 256 experts, which stream but for the short K: 2^23 + 2048 tiles of 256 columns, 2^24 + 4096 of 128."""
    dev, T, E, N = torch.device("cuda:0"), 65536, 256, 2048
    assert mb.moe_rows16_launch(mb.MOE_DTYPE_BF16, tile_n, T, E, E, K, N) == mb.MOE_ROWS16_PER_TILE_SMALL
    g = torch.Generator(device=dev).manual_seed(6)
    X = torch.randn(T, K, generator=g, device=dev).to(torch.bfloat16)
    W = (torch.randn(E, K, N, generator=g, device=dev) * K ** -0.5).to(torch.bfloat16)
    ids = torch.arange(E, dtype=torch.int32, device=dev).expand(T, E).contiguous()
    tmap = mb.alloc_task_map(T, E, E, 16, tile_n, N)
    mb.moe_build_task_map(ids, T, E, E, 16, tile_n, N, tmap)
    Y = torch.empty(T, E, N // 2, dtype=torch.bfloat16, device=dev)
    mb.moe_grouped_gemm(X, W, ids, tmap, Y, mb.GemmDesc(mb.MOE_DTYPE_BF16, T, E, E, K, N, 16, tile_n, epilogue=mb.MOE_EPILOGUE_SWIGLU))
    for e in (0, 1, 127, 128, 254, 255):
        gate, up = (X.double() @ W[e].double()).split(N // 2, dim=1)
        want = (torch.nn.functional.silu(gate) * up).to(torch.bfloat16).double()
        # as above: one bf16 rounding each, and K * 2^-24 of sums of at most about 4 * |x||w| (|w| of the order of 1 in all) in front of it
        assert ((Y[:, e].double() - want).abs() <= 2.0 ** -7 * want.abs() + 1e-4).all(), f"expert {e}"
