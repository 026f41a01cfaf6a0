"""The tail split at the sizes it is made for: every number of parts that a last round of 1 to 17 tiles per XCD gets, with and without
full rounds in front, ragged parts (a K that the parts do not divide), every task function, every order of the experts and more than 64 of
them, against 64-bit products; the blocks of the workspace that were written are those of the parts, with nothing outside it; tiles that do
not run in parts are bit for bit what moe_grouped_gemm gives.  And the layer plan that takes it."""
import pytest
import torch

from paper_2501_16103_amd import binding as mb
from tests import helpers as H
from tests.test_gpu_parity import _ids_from_counts

pytestmark = pytest.mark.gpu


CASES = [
    # tile_m (negative: 32 slack rows), rows per expert, n-tiles, K, order   tiles per XCD (the last XCDs may hold fewer)
    (256, [300, 1, 64], 2, 14336, 0),                 # 1: 8 parts of 28 k-tiles
    (256, [129, 256, 0, 513, 65], 3, 14336, 0),       # 3: 8 parts
    (-256, [288, 129, 200, 256, 31], 8, 9280, 0),     # 5: 6 parts of 24 and 25 k-tiles
    (256, [200, 100, 256], 16, 2560, 0),              # 6: 5 parts of 8 k-tiles
    (256, [200, 100, 90, 256], 16, 2304, 0),          # 8: 4 parts of 9 k-tiles
    (256, [200, 100, 90, 256], 16, 2112, 0),          # 8, K too short: half tiles
    (256, [70, 128, 250, 3, 1], 16, 7168, 0),         # 10: 3 parts of 37 and 38 k-tiles
    (256, [90, 128, 64, 250], 32, 6080, 0),           # 16: 2 parts of 47 and 48 k-tiles
    (256, [90, 128, 64, 250], 32, 5888, 0),           # 16, K too short for two parts: half tiles
    (-256, [288, 100, 257, 40], 34, 14336, 0),        # 17: whole
    (128, [128, 64, 129, 1], 7, 14336, 0),            # 128-row tiles, 5: 6 parts
    (128, [128, 64, 90, 1], 32, 9088, 0),             # 16: 2 parts of 71 k-tiles
    (128, [128, 64, 90, 1], 32, 8960, 0),             # 16, K too short for two parts: half tiles
    (64, [64, 33, 70], 2, 7168, 0),                   # 64-row tiles, 1: 8 parts
    (64, [64, 33, 70], 8, 2048, 0),                   # 64-row tiles have no halves: 4, 4 parts of 8 k-tiles
    (64, [64, 33, 64, 1], 32, 2304, 0),               # 16: 2 parts of 18 k-tiles
    (64, [64, 33, 64, 1], 32, 2176, 0),               # 16, K too short for two parts: whole
    (256, [9000, 1000], 8, 2304, 0),                  # 40: a full round and 8, 4 parts
    (-256, [9000, 280], 8, 7168, 0),                  # 37: a full round and 5, 6 parts
    (256, [700, 1, 60, 300, 90, 513], 5, 4096, 1),    # spread order, 7 of 11 m-tiles: 4 parts
    (-256, [2000, 1, 60, 300, 2, 600, 5], 5, 7168, 2),   # order by kind, an XCD's share of each
    (256, [1, 0, 3] * 30, 2, 6400, 0),                # 90 experts, 15: 2 parts of 50 k-tiles
    (128, [1, 0, 200] * 30, 1, 9216, 2),              # 90 experts, by kind
]


@pytest.mark.parametrize("tile_m,counts,nt,K,order", CASES)
def test_tail_parts(tile_m, counts, nt, K, order):
    dev = torch.device("cuda:0")
    slack, tile_m = (32, 256) if tile_m < 0 else (0, tile_m)
    E, T, N = len(counts), sum(counts), nt * 256
    ids = _ids_from_counts(counts, 5).to(dev)
    g = torch.Generator(device=dev).manual_seed(K + nt)
    X = torch.randn((T, K), generator=g, device=dev).to(torch.bfloat16)
    W = (torch.randn((E, K, N), generator=g, device=dev) * K ** -0.5).to(torch.bfloat16)
    tmap = mb.alloc_task_map(T, 1, E, tile_m, 256, N)
    mb.moe_build_task_map_ex(ids, T, 1, E, N, mb.Tiling(tile_m, 256, order, tile_m_slack=slack), tmap)
    desc = mb.GemmDesc(mb.MOE_DTYPE_BF16, T, 1, E, K, N, tile_m, 256, tile_m_slack=slack)
    words = mb.moe_tail_split_workspace_bytes(tile_m, 256) // 4
    guard, pad = 1024, 3
    buf = torch.full((words + 2 * guard,), float("nan"), dtype=torch.float32, device=dev)
    ws = buf[guard: guard + words]
    ybuf = torch.full((T + 2 * pad, N), float("nan"), dtype=torch.bfloat16, device=dev)
    Y, plain = ybuf[pad: pad + T], torch.full((T, N), float("nan"), dtype=torch.bfloat16, device=dev)
    mb.moe_grouped_gemm_tail_split(X, W, tmap, Y, desc, ws)
    mb.moe_grouped_gemm(X, W, None, tmap, plain, desc)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(Y.float()).all()), "an output was never written"
    assert bool(torch.isnan(ybuf[:pad].float()).all()) and bool(torch.isnan(ybuf[-pad:].float()).all()), "wrote outside Y"
    # one rounding to bf16 and fp32 sums in some order, against 64 bits
    for e in range(E):
        r = torch.nonzero(ids[:, 0] == e).flatten()
        for r in r.split(1024):
            want = X[r].double() @ W[e].double()
            bound = 2.0 ** -8 * want.abs() * 1.001 + H.sum_err_coeff(K, False) * (X[r].abs().double() @ W[e].abs().double()) + 1e-30
            assert bool(((Y[r].double() - want).abs() <= bound).all()), f"expert {e}"
    # which tiles ran in parts: slot s of XCD x runs block slots[x][s]
    total, heavy = int(tmap[mb.HDR["TOTAL_TILES"]]), int(tmap[18])   # header word 18: tiles of the heavy experts (order by kind)
    if order == 2:
        slots = []
        for x in range(8):
            h = list(range(heavy * x >> 3, heavy * (x + 1) >> 3))
            li = list(range(heavy + ((total - heavy) * x >> 3), heavy + ((total - heavy) * (x + 1) >> 3)))
            n = len(h) + len(li)   # the next light block whenever their share of the slots so far rises
            slots.append([li[s * len(li) // n] if (s + 1) * len(li) // n > s * len(li) // n else h[s - s * len(li) // n] for s in range(n)])
    else:
        share = -(-total // 8)
        slots = [list(range(min(x * share, total), min((x + 1) * share, total))) for x in range(8)]
    in_parts, blocks = set(), set()
    for x in range(8):
        t = len(slots[x]) % 32
        p = H.tail_parts(t, K // 64, tile_m)
        if p > 1:
            in_parts |= set(slots[x][len(slots[x]) - t:])
            blocks |= set(range(x * 32, x * 32 + t * p))
    # each part left its sums in the workspace, and nothing else was written there
    used = 256 * (tile_m + slack) * 256
    written = torch.isfinite(ws[:used].view(256, -1)).any(dim=1).nonzero().flatten().tolist()
    assert set(written) == blocks and not bool(torch.isfinite(ws[used:]).any()), "wrote to another block"
    assert bool(torch.isnan(buf[:guard]).all()) and bool(torch.isnan(buf[-guard:]).all()), "wrote outside the workspace"
    assert words == 256 * (288 if tile_m == 256 else tile_m) * 256, "32 blocks per XCD: the most that the parts of a round take"
    rows, B = [torch.nonzero(ids[:, 0] == e).flatten().tolist() for e in range(E)], 0
    sigma = tmap[mb.moe_map_offsets(E)["sigma"]:][:E].tolist()
    for e in sigma:
        if e < 0:
            break
        mt = max(1, -(-(counts[e] - slack) // tile_m))
        for n in range(nt):
            for m in range(mt):
                if B not in in_parts:
                    r = torch.tensor(rows[e][m * tile_m:] if m == mt - 1 else rows[e][m * tile_m:(m + 1) * tile_m], device=dev)
                    cols = slice(n * 256, (n + 1) * 256)
                    assert torch.equal(Y[r, cols].view(torch.int16), plain[r, cols].view(torch.int16)), f"tile {B}"
                B += 1
    assert B == total


@pytest.mark.parametrize("T,k,E,hidden,inter,tail", [(150, 2, 4, 256, 7168, True), (1, 2, 8, 512, 7168, True), (3, 2, 8, 256, 14336, True),
                                                     (1, 6, 64, 256, 384, False), (2, 2, 16, 512, 256, False)])
def test_layer_whose_down_product_leaves_the_default_tiling(T, k, E, hidden, inter, tail):
    """Layers whose down product takes the tail split (long K) or 128 x 128 tiles (a token or two): the down product is that of the
    layer's own activations, and its output their weighted sum."""
    dev = torch.device("cuda:0")
    plan = mb.MoeLayerPlan(T, k, E, hidden, inter, dev)
    assert plan.tail_split == tail and plan.k_parts == 1
    assert tail or (plan.g2.tile_m, plan.g2.tile_n) == (128, 128)
    g = torch.Generator(device=dev).manual_seed(3)
    X = torch.randn((T, hidden), generator=g, device=dev).to(torch.bfloat16)
    W1 = (torch.randn((E, hidden, 2 * inter), generator=g, device=dev) * hidden ** -0.5).to(torch.bfloat16)
    W2 = (torch.randn((E, inter, hidden), generator=g, device=dev) * inter ** -0.5).to(torch.bfloat16)
    ids = torch.stack([torch.randperm(E, generator=g, device=dev)[:k] for _ in range(T)]).to(torch.int32)
    wts = torch.rand((T, k), generator=g, device=dev, dtype=torch.float32)
    if tail:
        plan.workspace.fill_(float("nan"))
    out = plan.forward(X, W1, W2, ids, wts)
    torch.cuda.synchronize()
    flat, act = ids.reshape(-1).long(), plan.act
    for e in range(E):
        r = torch.nonzero(flat == e).flatten()
        want = act[r].double() @ W2[e].double()
        bound = 2.0 ** -8 * want.abs() * 1.001 + H.sum_err_coeff(inter, False) * (act[r].abs().double() @ W2[e].abs().double()) + 1e-30
        assert bool(((plan.down[r].double() - want).abs() <= bound).all())
    terms = plan.down.double().view(T, k, hidden) * wts.double()[:, :, None]
    want = terms.sum(dim=1)
    bound = 2.0 ** -8 * want.abs() * 1.001 + (k + 1) * 2.0 ** -24 * terms.abs().sum(dim=1) + 1e-30
    assert bool(((out.double() - want).abs() <= bound).all())
