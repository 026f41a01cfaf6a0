"""The calls whose time counts, over the sizes that this library is used at.

Two kinds of call, both as a serving program makes them once per step and layer, with every buffer and plan already
in hand and the routing of the step as the new input:

  "product"  moe_build_task_map_ex, then moe_grouped_gemm: one projection of all experts;
  "layer"    MoeLayerPlan.forward: map, gate+up product with the fused activation, map, down product (along K in parts
             where the plan says so), weighted sum.

Sizes are those of the repository's own workloads: the fp8 decode layer (64 experts, top-6, 2048 -> 2816) and the same
layer in bf16, the Mixtral-shaped experts (8, top-2, 4096 / 14336), the fine-grained ones (256, top-8, 7168 -> 4096)
and the evaluation of Sec. 5 of the paper (64 experts, top-8, [3584, 2560]).
"""
import math

import torch

from paper_2501_16103_amd import binding as mb

# K -> N of one projection ("product") or hidden / intermediate size ("layer"), experts, top-k
SHAPES = {
    "fp8_expert": dict(kind="product", dtype="fp8", E=64, k=6, K=2048, N=2816),
    "mixtral_up": dict(kind="product", dtype="bf16", E=8, k=2, K=4096, N=28672),
    "fine_grained": dict(kind="product", dtype="bf16", E=256, k=8, K=7168, N=4096),
    "paper_eval": dict(kind="product", dtype="bf16", E=64, k=8, K=3584, N=2560),
    "small_layer": dict(kind="layer", dtype="bf16", E=64, k=6, hidden=2048, inter=1408),
    "mixtral_layer": dict(kind="layer", dtype="bf16", E=8, k=2, hidden=4096, inter=14336),
}
E4M3_MAX = 448.0


def _case(family, T, routing="gauss", layout="kn", swiglu=False):
    return dict(family=family, T=T, routing=routing, layout=layout, swiglu=swiglu)


def listed():
    def c(name, *a, **kw):
        return dict(_case(*a, **kw), name=name)
    return [
        # generating one sequence, one token per step: launches and latency
        c("fp8_decode_T1", "fp8_expert", 1),
        c("small_layer_T1", "small_layer", 1),
        # generating a batch of sequences: every expert's weights are read for a few tokens each
        c("fp8_decode_T32", "fp8_expert", 32),
        c("mixtral_layer_T16", "mixtral_layer", 16),
        # a large decoding batch or a short prompt, with the uneven expert loads of a trained router
        c("mixtral_layer_zipf_T333", "mixtral_layer", 333, routing="zipf"),
        c("small_layer_T777", "small_layer", 777),
        # many small experts, about thirty tokens each: weights dominate, but tiles are no longer nearly empty
        c("fine_grained_T1000", "fine_grained", 1000),
        # prompts: compute-bound; the fp8 one with its activation fused, as the gate+up projection is called
        c("fp8_prefill_swiglu_T4096", "fp8_expert", 4096, swiglu=True),
        c("mixtral_up_T4096", "mixtral_up", 4096),
        c("mixtral_layer_T4096", "mixtral_layer", 4096),
        # weights in the order in which linear layers are stored, [E][N][K]
        c("mixtral_up_nk_T2047", "mixtral_up", 2047, layout="nk"),
        # the paper's uneven scenario: eight experts with nearly all tokens, 56 with one token each
        c("paper_eval_worst", "paper_eval", 4096, routing="worst"),
    ]


def draw(rng):
    family, lo, hi = rng.choice([("fp8_expert", 1, 256), ("fp8_expert", 257, 8192), ("small_layer", 1, 8192),
                                 ("mixtral_layer", 1, 4096), ("mixtral_up", 512, 4096), ("fine_grained", 16, 1200),
                                 ("paper_eval", 1024, 4096)])
    T = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    T = min(max(T, lo), hi)
    routing, layout, swiglu = "gauss", "kn", False
    if family == "fp8_expert":
        if T <= 256:
            layout = rng.choice(["kn", "kn", "nk"])   # (fp8 kernels for [E][N][K] weights exist for the 16-row tiles)
        swiglu = rng.random() < 0.5
    elif family == "mixtral_up":
        layout = rng.choice(["kn", "nk"])
        swiglu = rng.random() < 0.5
    elif family == "paper_eval":
        routing = rng.choice(["balanced", "best", "worst"])
    elif family != "fine_grained":
        routing = rng.choice(["gauss", "zipf"])
    return _case(family, T, routing, layout, swiglu)


# ---------------------------------------------------------------- inputs

def _device():
    return torch.device("cuda:0")


def _gen(seed, tag):
    g = torch.Generator(device=_device())
    g.manual_seed((int(seed) * 1000003 + tag) % (1 << 62))
    return g


def _routing(case, seed):
    """int32 [T, k] distinct experts per token, fp32 [T, k] router weights."""
    s, T = SHAPES[case["family"]], case["T"]
    E, k, dev, g = s["E"], s["k"], _device(), _gen(seed, 1)
    logits = torch.randn(T, E, generator=g, device=dev)
    perm = torch.randperm(E, generator=g, device=dev)      # which experts are the busy ones
    if case["routing"] == "gauss":
        top = torch.topk(logits, k, dim=1)
        ids, val = top.indices, top.values
    elif case["routing"] == "zipf":
        # k draws without replacement from p ~ rank^-1.2 (the largest of log p + Gumbel noise)
        u = torch.rand(T, E, generator=g, device=dev).clamp_(1e-12, 1 - 1e-7)
        logp = -1.2 * torch.log(torch.arange(1, E + 1, device=dev, dtype=torch.float32))
        top = torch.topk(logp - torch.log(-torch.log(u)), k, dim=1)
        ids, val = perm[top.indices], top.values
    else:
        val = logits[:, :k]
        if case["routing"] == "balanced":
            ids = torch.arange(T * k, device=dev).reshape(T, k) % E
        else:
            ids = torch.arange(k, device=dev).expand(T, k).clone()
            if case["routing"] == "worst":
                n = min(E - k, T)
                ids[:n, k - 1] = k + torch.arange(n, device=dev)
        ids = perm[ids][torch.randperm(T, generator=g, device=dev)]
    return ids.to(torch.int32).contiguous(), torch.softmax(val, dim=1).contiguous()


def _weights(shape, K, fp8, seed, tag):
    """N(0, 1/K) of shape [E, ., .]; fp8: e4m3 bytes and one scale per expert."""
    W = torch.empty(shape, dtype=torch.uint8 if fp8 else torch.bfloat16, device=_device())
    scale = torch.empty(shape[0], dtype=torch.float32, device=_device()) if fp8 else None
    g = _gen(seed, tag)
    for e in range(shape[0]):
        if not fp8:
            W[e].normal_(0.0, K ** -0.5, generator=g)
            continue
        w = torch.randn(shape[1:], generator=g, device=_device()) * (K ** -0.5)
        scale[e] = w.abs().amax() / E4M3_MAX
        W[e] = (w / scale[e]).to(torch.float8_e4m3fn).view(torch.uint8)
    return W, scale


def _tokens(T, K, fp8, seed):
    x = torch.randn(T, K, generator=_gen(seed, 2), device=_device())
    if not fp8:
        return x.to(torch.bfloat16), None
    scale = x.abs().amax(dim=1) / E4M3_MAX
    return (x / scale[:, None]).to(torch.float8_e4m3fn).view(torch.uint8), scale


def _inputs(case, seed):
    s, T = SHAPES[case["family"]], case["T"]
    ids, topw = _routing(case, seed)
    if s["kind"] == "layer":
        h, i, E = s["hidden"], s["inter"], s["E"]
        return dict(ids=ids, topw=topw, X=_tokens(T, h, False, seed)[0], W1=_weights((E, h, 2 * i), h, False, seed, 3)[0],
                    W2=_weights((E, i, h), i, False, seed, 4)[0])
    K, N, fp8 = s["K"], s["N"], s["dtype"] == "fp8"
    X, xs = _tokens(T, K, fp8, seed)
    W, ws = _weights((s["E"], N, K) if case["layout"] == "nk" else (s["E"], K, N), K, fp8, seed, 3)
    return dict(ids=ids, X=X, xs=xs, W=W, ws=ws)


def prepare(case, seed):
    s, T = SHAPES[case["family"]], case["T"]
    st = _inputs(case, seed)
    if s["kind"] == "layer":
        st["plan"] = mb.MoeLayerPlan(T, s["k"], s["E"], s["hidden"], s["inter"], _device())
        return st
    K, N, E, k = s["K"], s["N"], s["E"], s["k"]
    dtype = mb.MOE_DTYPE_FP8_E4M3 if s["dtype"] == "fp8" else mb.MOE_DTYPE_BF16
    layout = mb.MOE_W_LAYOUT_NK if case["layout"] == "nk" else mb.MOE_W_LAYOUT_KN
    g = mb.moe_default_tiling(dtype, T, k, E, K, N)
    if not mb.moe_w_layout_supported(dtype, g, layout):
        g = mb.Tiling(256, 256)
    st["tiling"] = g
    st["map"] = mb.alloc_task_map(T, k, E, g.tile_m, g.tile_n, N, _device())
    st["Y"] = torch.empty((T, k, N // 2 if case["swiglu"] else N), dtype=torch.bfloat16, device=_device())
    st["desc"] = mb.GemmDesc(dtype, T, k, E, K, N, g.tile_m, g.tile_n, st["xs"], st["ws"], tile_m_slack=g.tile_m_slack,
                             epilogue=mb.MOE_EPILOGUE_SWIGLU if case["swiglu"] else mb.MOE_EPILOGUE_NONE, w_layout=layout)
    return st


def run(st):
    if "plan" in st:
        return st["plan"].forward(st["X"], st["W1"], st["W2"], st["ids"], st["topw"])
    d = st["desc"]
    mb.moe_build_task_map_ex(st["ids"], d.T, d.k, d.E, d.N, st["tiling"], st["map"])
    mb.moe_grouped_gemm(st["X"], st["W"], st["ids"], st["map"], st["Y"], d)
    return st["Y"]


# ---------------------------------------------------------------- what a pass cannot do without

def _touched(case):
    """Experts with at least one token (expected number)."""
    s, T = SHAPES[case["family"]], case["T"]
    E, k = s["E"], s["k"]
    if case["routing"] == "gauss":
        return E * (1.0 - (1.0 - k / E) ** T)
    if case["routing"] == "zipf":
        p = [r ** -1.2 for r in range(1, E + 1)]
        total = sum(p)
        return max(float(k), sum(1.0 - (1.0 - q / total) ** (k * T) for q in p))
    if case["routing"] == "balanced":
        return min(E, T * k)
    return k + (min(E - k, T) if case["routing"] == "worst" else 0)


def work(case):
    s, T = SHAPES[case["family"]], case["T"]
    R, n = T * s["k"], _touched(case)
    if s["kind"] == "layer":
        h, i = s["hidden"], s["inter"]
        return {"bytes": 2.0 * (3 * n * h * i + 2 * T * h) + 8.0 * R, "flops": 2.0 * R * 3 * h * i}
    K, N, es = s["K"], s["N"], 1 if s["dtype"] == "fp8" else 2
    out = N // 2 if case["swiglu"] else N
    scales = 4.0 * (T + n) if s["dtype"] == "fp8" else 0.0
    return {"bytes": es * (n * K * N + T * K) + 2.0 * R * out + 4.0 * R + scales, "flops": 2.0 * R * K * N}


def tolerance(case):
    # One rounding of an fp32 sum to bf16 is 1.7e-3 in the 2-norm, two correct sums differ where they round apart.
    # A layer rounds three times (activation, down product, sum).
    return {"rel": 7e-3, "max": 2e-2} if SHAPES[case["family"]]["kind"] == "product" else {"rel": 1e-2, "max": 4e-2}


# ---------------------------------------------------------------- the same in 64 bits

def _by_expert(rows, ids, E, product, width):
    """out[r] = product(rows of expert e, e) for every routed row r (flat order t * k + j)."""
    flat = ids.reshape(-1).long()
    out = torch.empty((flat.numel(), width), dtype=torch.float64, device=_device())
    for e in range(E):
        r = torch.nonzero(flat == e).flatten()
        if r.numel():
            out[r] = product(rows(r), e)
    return out


def _silu_mul(gu):
    half = gu.shape[1] // 2
    g = gu[:, :half]
    return g / (1.0 + torch.exp(-g)) * gu[:, half:]


def exact(case, seed):
    s, T = SHAPES[case["family"]], case["T"]
    E, k = s["E"], s["k"]
    st = _inputs(case, seed)
    ids, X = st["ids"], st["X"]
    if s["kind"] == "layer":
        X = X.double()
        act = _by_expert(lambda r: X[r // k], ids, E, lambda x, e: _silu_mul(x @ st["W1"][e].double()), s["inter"])
        down = _by_expert(lambda r: act[r], ids, E, lambda x, e: x @ st["W2"][e].double(), s["hidden"])
        return (down.reshape(T, k, -1) * st["topw"].double()[:, :, None]).sum(dim=1)

    def value(t):
        return t.view(torch.float8_e4m3fn).float().double() if s["dtype"] == "fp8" else t.double()

    X = value(X) * (st["xs"].double()[:, None] if st["xs"] is not None else 1.0)

    def product(x, e):
        w = value(st["W"][e])
        y = x @ (w.t() if case["layout"] == "nk" else w)
        if st["ws"] is not None:
            y = y * st["ws"][e].double()
        return _silu_mul(y) if case["swiglu"] else y

    width = s["N"] // 2 if case["swiglu"] else s["N"]
    return _by_expert(lambda r: X[r // k], ids, E, product, width).reshape(T, k, width)
