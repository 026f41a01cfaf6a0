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


# ---- the deep instructions' error against 64 bits

def _e4m3(x):
    return x.clamp(-448, 448).to(torch.float8_e4m3fn)


def _error_inputs(kind, T, K, N, g, dev):
    """X [T, K], W [K, N] (float, before the cast).  Magnitudes: e4m3's whole range, evenly spread over its exponents.  cancelN:
    every product occurs once with either sign, both within the same N consecutive k, so the exact sums are 0 and what comes
    out is the error alone.  huge: small positive terms and, in every 128, one pair of +-448 * 448 within 32 of them."""
    def spread(*s):
        r = torch.rand((2,) + s, generator=g, device=dev)
        return torch.exp2(r[0] * 17 - 9) * torch.sign(r[1] - 0.5)
    if kind == "normal":
        return torch.randn(T, K, generator=g, device=dev) * 100, torch.randn(K, N, generator=g, device=dev) * 100
    if kind == "spread":
        return spread(T, K), spread(K, N)
    if kind == "huge":
        X, W = (0.5 * (1 + torch.rand(*s, generator=g, device=dev)) for s in ((T, K), (K, N)))
        for b in range(96, K, 128):
            X[:, b] = X[:, b + 31] = W[b] = 448.0
            W[b + 31] = -448.0
        return X, W
    n = K if kind == "cancel" else int(kind[6:])
    order = torch.randperm(K, generator=g, device=dev) if kind == "cancel" else torch.arange(K, device=dev)
    X, W = torch.empty(T, K, device=dev), torch.empty(K, N, device=dev)
    half = order.reshape(K // n, 2, n // 2)
    x, w = spread(T, K // 2), spread(K // 2, N)
    for h, sign in ((0, 1.0), (1, -1.0)):
        X[:, half[:, h].reshape(-1)], W[half[:, h].reshape(-1)] = x, sign * w
    return X, W


@pytest.mark.parametrize("K", [128, 1024, 8192])
@pytest.mark.parametrize("kind", ["normal", "spread", "cancel", "cancel32", "cancel64", "cancel128", "huge"])
def test_deep_instruction_error(dev, kind, K):
    """The sums of the 256-, 128- and 64-row functions (16x16x128 and 32x32x64) stay within the adder's bound, and their error
    is no larger than that of the 16-row tiles, which use 16x16x32 (measured: the same to every digit)."""
    T, N = 256, 256
    g = torch.Generator(device=dev).manual_seed(K)
    X, W = (_e4m3(t) for t in _error_inputs(kind, T, K, N, g, dev))
    Xd, Wd = X.double().cpu(), W.double().cpu()     # (products and their sums are exact in 64 bits)
    exact, A, limit = (Xd @ Wd).to(dev), (Xd.abs() @ Wd.abs()).to(dev), H.fp8_adder_bound(X.float(), W.float())

    def error(rows, tile_m):
        tmap = mb.alloc_task_map(rows, 1, 1, tile_m, 256, N, dev)
        mb.moe_build_task_map(torch.zeros(rows, 1, dtype=torch.int32, device=dev), rows, 1, 1, tile_m, 256, N, tmap)
        Y, one = torch.full((rows, N), float("nan"), dtype=torch.bfloat16, device=dev), torch.ones(rows, device=dev)
        mb.moe_grouped_gemm(X[:rows].contiguous().view(torch.uint8), W[None].contiguous().view(torch.uint8), None, tmap, Y,
                            mb.GemmDesc(mb.MOE_DTYPE_FP8_E4M3, rows, 1, 1, K, N, tile_m, 256, one, one[:1].clone()))
        return (Y.double() - exact[:rows]).abs()

    for rows, tile_m in ((256, 256), (128, 256), (64, 256), (256, 64)):
        err, shallow = error(rows, tile_m), error(rows, 16)
        a, bound = A[:rows], limit[:rows]
        assert (err <= bound + 2.0 ** -8 * (exact[:rows].abs() + bound)).all(), (rows, tile_m)     # (+ the rounding to bf16)
        for what in (lambda e: (e / a).max(), lambda e: ((e / a) ** 2).mean().sqrt()):
            assert what(err) <= 1.02 * what(shallow) + 1e-12, (rows, tile_m, float(what(err)), float(what(shallow)))


@pytest.mark.parametrize("ratio,same,other", [(13, True, True), (14, False, True), (22, False, True)])
def test_fp8_adder_groups(dev, ratio, same, other):
    """What fp8_adder_bound rests on: beside +-2^16, a product of 2^(16 - ratio) in the same 8 k and in the next 8, for the
    three instructions."""
    K, N = 128, 256
    for tile_m in (16, 64, 256):
        T = tile_m
        for at, kept in ((5, same), (8 + 5, other)):
            X, W = torch.zeros(T, K, device=dev), torch.zeros(K, N, device=dev)
            X[:, 0], X[:, 3], W[0], W[3] = 256.0, 256.0, 256.0, -256.0
            ex = (16 - ratio + 1) // 2
            X[:, at], W[at] = 2.0 ** ex, 2.0 ** (16 - ratio - ex)
            tmap = mb.alloc_task_map(T, 1, 1, tile_m, 256, N, dev)
            mb.moe_build_task_map(torch.zeros(T, 1, dtype=torch.int32, device=dev), T, 1, 1, tile_m, 256, N, tmap)
            Y, one = torch.full((T, N), float("nan"), dtype=torch.bfloat16, device=dev), torch.ones(T, device=dev)
            mb.moe_grouped_gemm(_e4m3(X).view(torch.uint8), _e4m3(W)[None].contiguous().view(torch.uint8), None, tmap, Y,
                                mb.GemmDesc(mb.MOE_DTYPE_FP8_E4M3, T, 1, 1, K, N, tile_m, 256, one, one[:1].clone()))
            want = 2.0 ** (16 - ratio) if kept else 0.0
            assert (Y.double() == want).all(), (tile_m, at, float(Y[0, 0]), want)
