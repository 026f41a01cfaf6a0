"""A step of a few rows: the maps of a layer and its first product in one launch, against the two calls."""
import numpy as np
import pytest
import torch

from paper_2501_16103_amd import binding as mb

pytestmark = pytest.mark.gpu

# the forms of the one launch, for 128- and 256-wide tiles (None: the two calls' launches)
TILE, DEEP, PAIRS, STREAM = mb.MOE_ROWS16_PER_TILE, mb.MOE_ROWS16_PER_TILE_DEEP, mb.MOE_ROWS16_PAIRS, mb.MOE_ROWS16_STREAM


def _routing(kind, T, k, E, g):
    if kind == "one":          # every row on one expert: several 16-row tiles, rows beyond the first in the same lane order
        return torch.full((T, k), E - 1, dtype=torch.int32)
    if kind == "repeat":       # ids drawn with repetition, also within a token
        return torch.randint(0, E, (T, k), generator=g, dtype=torch.int32)
    if kind == "bad":
        ids = torch.randint(0, E, (T, k), generator=g, dtype=torch.int32)
        ids[T // 2, k - 1] = E
        return ids
    return torch.stack([torch.randperm(E, generator=g)[:k] for _ in range(T)]).to(torch.int32)


@pytest.mark.parametrize("T,k,E,K,N,kind,swiglu,forms", [
    (1, 6, 64, 256, 384, "topk", True, (TILE,)),        # 128-wide tiles, one workgroup each
    (1, 1, 1, 192, 256, "topk", False, (TILE, DEEP)),        # the smallest K and one expert
    (7, 2, 8, 512, 640, "topk", False, (TILE,)),        # N with an odd number of 128-wide tiles
    (64, 1, 64, 256, 2816, "topk", True, (PAIRS, STREAM)),      # as many rows and experts as a wavefront has lanes
    (10, 6, 64, 320, 2816, "repeat", True, (PAIRS, STREAM)),    # 256-wide tiles or pairs, resident
    (32, 2, 5, 256, 512, "repeat", False, (TILE, DEEP)),
    (33, 1, 3, 256, 256, "one", False, (TILE, DEEP)),        # three tiles of one expert, the last with one row
    (64, 1, 64, 256, 128, "one", True, (TILE,)),
    (4, 6, 64, 2048, 2816, "topk", True, (PAIRS, DEEP)),      # 256-wide tiles, one workgroup each
    (9, 7, 60, 256, 8192, "topk", False, (PAIRS, STREAM)),      # 63 rows, E below a multiple of 64
    (12, 5, 64, 256, 512, "bad", False, (TILE, DEEP)),       # an id outside [0, E): maps with a status, no product
    (13, 5, 64, 256, 512, "topk", False, (None, None)),      # 65 rows: the two calls
    (6, 4, 65, 256, 512, "topk", False, (None, None)),       # 65 experts: the two calls
])
def test_product_with_its_maps(T, k, E, K, N, kind, swiglu, forms):
    dev = torch.device("cuda:0")
    g = torch.Generator().manual_seed(100 * T + E)
    ids = _routing(kind, T, k, E, g).to(dev)
    X = torch.randn((T, K), generator=g).to(torch.bfloat16).to(dev)
    W = (torch.randn((E, K, N), generator=g) * K ** -0.5).to(torch.bfloat16).to(dev)
    out = N // 2 if swiglu else N
    assert len(forms) == sum(N % tile_n == 0 for tile_n in (128, 256))
    for tile_n, form in zip((128, 256), forms):
        g1, g2, N2 = mb.Tiling(16, tile_n), mb.Tiling(128, 128), 256
        d = mb.GemmDesc(mb.MOE_DTYPE_BF16, T, k, E, K, N, 16, tile_n, epilogue=int(swiglu))
        assert mb.moe_pair_gemm_launches(T, k, E, N, g1, d) == (1 if form else 2)
        assert form is None or mb.moe_rows16_launch(mb.MOE_DTYPE_BF16, tile_n, T, k, E, K, N) == form
        got = []
        for together in (False, True):
            m1, m2 = mb.alloc_task_map(T, k, E, 16, tile_n, N, dev), mb.alloc_task_map(T * k, 1, E, 128, 128, N2, dev)
            m1.fill_(-7), m2.fill_(-7)
            Y = torch.full((T * k, out), 9.0, dtype=torch.bfloat16, device=dev)
            if together:
                mb.moe_build_task_map_pair_gemm(ids, T, k, E, N, g1, m1, N2, g2, m2, X, W, Y, d)
            else:
                mb.moe_build_task_map_pair(ids, T, k, E, N, g1, m1, N2, g2, m2)
                mb.moe_grouped_gemm(X, W, ids, m1, Y, d)
            torch.cuda.synchronize()
            got.append((m1.cpu(), m2.cpu(), Y.view(torch.int16).cpu()))
        for a, b in zip(*got):
            assert torch.equal(a, b)
        assert mb.moe_task_map_status(m1) == (mb.MOE_ERR_ROUTING if kind == "bad" else mb.MOE_OK)
        if kind == "bad":
            assert bool((Y == 9.0).all())
        else:
            if T * k * K * N >= 1 << 28:
                continue
            want = torch.einsum("rk,rkn->rn", X.float().repeat_interleave(k, 0), W[ids.flatten().long()].float())
            if swiglu:
                want = torch.nn.functional.silu(want[:, :out]) * want[:, out:]
            err = (Y.float() - want).abs()
            assert float(err.max()) < 2.0 ** -7 * float(want.abs().max()) + 1e-3
            assert np.isfinite(float(err.max()))


def test_product_with_its_maps_refuses_what_the_calls_refuse():
    dev = torch.device("cuda:0")
    T, k, E, K, N = 2, 2, 8, 256, 256
    ids = torch.zeros((T, k), dtype=torch.int32, device=dev)
    X = torch.zeros((T, K), dtype=torch.bfloat16, device=dev)
    W = torch.zeros((E, K, N), dtype=torch.bfloat16, device=dev)
    Y = torch.zeros((T * k, N), dtype=torch.bfloat16, device=dev)
    g1, g2 = mb.Tiling(16, 128), mb.Tiling(128, 128)
    m1, m2 = mb.alloc_task_map(T, k, E, 16, 128, N, dev), mb.alloc_task_map(T * k, 1, E, 128, 128, N, dev)
    d = mb.GemmDesc(mb.MOE_DTYPE_BF16, T, k, E, K, N, 16, 128)

    def call(maps=(m1, m2), X=X, Y=Y, d=d):
        return mb.moe_build_task_map_pair_gemm(ids, T, k, E, N, g1, maps[0], N, g2, maps[1], X, W, Y, d, check=False)
    assert call() == mb.MOE_OK
    assert call(maps=(m1, m1)) == mb.MOE_ERR_INVALID_ARG                       # maps that overlap
    assert call(X=None) == mb.MOE_ERR_INVALID_ARG
    assert call(Y=Y.flatten()[1:]) == mb.MOE_ERR_INVALID_ARG                   # two bytes off a 16-byte boundary
    assert call(d=mb.GemmDesc(mb.MOE_DTYPE_BF16, T, k, E, 200, N, 16, 128)) == mb.MOE_ERR_UNSUPPORTED
    assert call(d=mb.GemmDesc(mb.MOE_DTYPE_BF16, T, k, E, K, N, 16, 128, launch_mode=-1)) == mb.MOE_ERR_INVALID_ARG
    torch.cuda.synchronize()


def test_layer_of_a_few_rows_replays_from_a_graph():
    """The launch takes the ids of each replay, not those of the capture, and its maps are rewritten each time."""
    dev = torch.device("cuda:0")
    T, k, E, hidden, inter = 3, 2, 32, 256, 256
    g = torch.Generator(device=dev).manual_seed(8)
    X = torch.randn((T, hidden), generator=g, device=dev).to(torch.bfloat16)
    W1 = (torch.randn((E, hidden, 2 * inter), generator=g, device=dev) * hidden ** -0.5).to(torch.bfloat16)
    W2 = (torch.randn((E, inter, hidden), generator=g, device=dev) * inter ** -0.5).to(torch.bfloat16)
    wts = torch.rand((T, k), generator=g, device=dev, dtype=torch.float32)
    plan, eager = mb.MoeLayerPlan(T, k, E, hidden, inter, dev), mb.MoeLayerPlan(T, k, E, hidden, inter, dev)
    assert plan.g1.tile_m == 16
    ids = torch.zeros((T, k), dtype=torch.int32, device=dev)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        plan.forward(X, W1, W2, ids, wts)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            plan.forward(X, W1, W2, ids, wts)
    for it in range(4):
        ids.copy_(torch.stack([torch.randperm(E, generator=g, device=dev)[:k] for _ in range(T)]))
        X.normal_(generator=g)
        want = eager.forward(X, W1, W2, ids, wts).clone()
        plan.out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(plan.out.view(torch.int16), want.view(torch.int16)), f"replay {it}"
        for m, want_m in ((plan.map1, eager.map1), (plan.map2, eager.map2)):
            written = mb.moe_map_offsets(E)["sorted_rows"] + T * k      # (words: header to the token index arrays)
            assert torch.equal(m[:written], want_m[:written])
