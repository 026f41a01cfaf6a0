"""A layer whose gate+up product the plan gives to the streaming launch, against 64-bit sums on the device."""
import pytest
import torch

from paper_2501_16103_amd import binding as mb

pytestmark = pytest.mark.gpu


def _routing(kind, T, k, E, g, dev):
    if kind == "even":
        return torch.stack([torch.randperm(E, generator=g, device=dev)[:k] for _ in range(T)]).to(torch.int32)
    if kind == "few":          # k experts with all rows: several tiles of 64 rows each, the others empty
        return torch.tensor([[E - 1, 2, 0, 5][:k]], dtype=torch.int32, device=dev).expand(T, k).contiguous()
    ids = torch.randint(1, E, (T, k), generator=g, device=dev, dtype=torch.int32)      # one with half of them
    ids[:, 0] = 0
    return ids


@pytest.mark.parametrize("kind", ["even", "few", "half"])
@pytest.mark.parametrize("T,k,E,hidden,inter", [
    (64, 2, 8, 1024, 7168),      # 448 wide tiles, merged for the round it saves; the shortest K
    (67, 4, 16, 1152, 7168),     # 896, 17 rows per expert, a K of 18 k-tiles
    (191, 2, 24, 1024, 3072),    # 576, the most rows for as many experts
])
def test_streamed_layer(kind, T, k, E, hidden, inter):
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(T)
    plan = mb.MoeLayerPlan(T, k, E, hidden, inter, dev)
    assert (plan.g1.tile_m, plan.g1.tile_n) == (16, 256)
    assert mb.moe_rows16_launch(mb.MOE_DTYPE_BF16, 256, T, k, E, hidden, 2 * inter) == mb.MOE_ROWS16_STREAM_MERGED
    ids, wts = _routing(kind, T, k, E, g, dev), torch.rand((T, k), generator=g, device=dev)
    X = torch.randn((T, hidden), generator=g, device=dev).to(torch.bfloat16)
    W1 = (torch.randn((E, hidden, 2 * inter), generator=g, device=dev) * hidden ** -0.5).to(torch.bfloat16)
    W2 = (torch.randn((E, inter, hidden), generator=g, device=dev) * inter ** -0.5).to(torch.bfloat16)
    plan.act.fill_(float("nan"))
    out = plan.forward(X, W1, W2, ids, wts).double()
    act, down, flat = plan.act.view(T * k, inter), plan.down.view(T * k, hidden), ids.flatten().long()
    for e in range(E):
        r = torch.nonzero(flat == e).flatten()
        if r.numel() == 0:
            continue
        gate, up = (X[r // k].double() @ W1[e].double()).split(inter, dim=1)
        want = torch.nn.functional.silu(gate) * up
        # one rounding to bf16 (2^-9 relative), and fp32 sums of K products of size |x||w| ~ K^-1/2: K * 2^-24 * K^-1/2, on both factors (at most about 5)
        assert ((act[r].double() - want).abs() <= 2.0 ** -8 * want.abs() + 10 * hidden ** 0.5 * 2.0 ** -24 + 2.0 ** -30).all(), f"act, expert {e}"
        want = act[r].double() @ W2[e].double()
        assert ((down[r].double() - want).abs() <= 2.0 ** -8 * want.abs() + 10 * inter ** 0.5 * 2.0 ** -24).all(), f"down, expert {e}"
    want = (down.view(T, k, hidden).double() * wts.double()[:, :, None]).sum(dim=1)
    assert ((out - want).abs() <= 2.0 ** -8 * want.abs() + 1e-6).all()
