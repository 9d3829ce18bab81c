"""What a user of this library has it do, as timed cases: pruning and packing a layer or a whole model, the
hybrid-sparse product on its own, single convolutions and the chained ResNet-50 forward, from calls of a few
microseconds to milliseconds.

A case is a dict of plain values; its "kind" says which entry points it goes through:
  prune   prune_and_pack (crisp_select_pack) of one layer
  model   crisp_select_pack_batch over the 53 convolutions of ResNet-50
  gemm    crisp_spmm, or crisp_spmm_ep when the layer tail (scale, bias, residual, ReLU) is fused in
  conv    conv_forward: a convolution by the way the library plans for it
  net     resnet.forward: the 53 convolutions chained, with max-pool, shortcuts and layer tails
Products read layers that were pruned and packed beforehand, as a served model has them.
"""
import math

import torch

from paper_2311_14272_amd import crisp, resnet, synth

PATTERNS = ((1, 4), (2, 4), (3, 4), (1, 8), (2, 8), (4, 8))


def listed():
    return [
        # one small layer pruned by itself: the 256 x 1024 1x1 layer of a bottleneck at 14x14
        {"name": "prune_layer", "kind": "prune", "S": 256, "K": 1024, "n": 1, "m": 4, "B": 64, "d": 0.3, "sal": 1, "topk": 0},
        # one-shot pruning of a whole model (gradient saliency), all layers in one call
        {"name": "prune_resnet50", "kind": "model", "B": 64, "plan": 0},
        # a 3x3 layer of a single image, lowered beforehand: the smallest product, fp32 out
        {"name": "gemm_small_b32", "kind": "gemm", "S": 256, "K": 1152, "N": 3136, "n": 2, "m": 4, "B": 32, "d": 0.5,
         "bf16": 0, "ep": 0, "res": 0, "k8": 0, "topk": 0},
        # a pointwise layer of a mobile network: few channels, very many positions
        {"name": "gemm_pointwise_b32", "kind": "gemm", "S": 24, "K": 144, "N": 401408, "n": 2, "m": 4, "B": 32, "d": 0.6,
         "bf16": 1, "ep": 0, "res": 0, "k8": 0, "topk": 0},
        # a large lowered 3x3 layer (512 -> 512 channels at 28x28, batch 64): long block-rows
        {"name": "gemm_large_2of8", "kind": "gemm", "S": 512, "K": 4608, "N": 50176, "n": 2, "m": 8, "B": 64, "d": 0.25,
         "bf16": 1, "ep": 0, "res": 0, "k8": 0, "topk": 0},
        # a 1x1 layer with the densest of the benchmark's patterns (not a two-of-four one)
        {"name": "gemm_1x1_4of8", "kind": "gemm", "S": 512, "K": 1024, "N": 50176, "n": 4, "m": 8, "B": 64, "d": 0.5,
         "bf16": 1, "ep": 0, "res": 0, "k8": 0, "topk": 0},
        # a channel-expanding 1x1 layer with its whole tail: folded normalisation, shortcut, ReLU
        {"name": "gemm_expand_tail", "kind": "gemm", "S": 1024, "K": 256, "N": 50176, "n": 2, "m": 4, "B": 64, "d": 0.5,
         "bf16": 1, "ep": 1, "res": 1, "k8": 0, "topk": 0},
        # nothing divides anything: odd channel count, K and number of columns
        {"name": "gemm_ragged", "kind": "gemm", "S": 203, "K": 459, "N": 25003, "n": 2, "m": 4, "B": 32, "d": 0.5,
         "bf16": 1, "ep": 1, "res": 0, "k8": 0, "topk": 0},
        # the 3x3 layer of a bottleneck at 14x14, batch 256
        {"name": "conv3x3_14", "kind": "conv", "S": 256, "C": 256, "H": 14, "batch": 256, "k": 3, "stride": 1, "n": 2, "m": 8,
         "B": 64, "d": 0.6, "bf16": 1, "ep": 1},
        # the 3x3 layer that halves the resolution from 14x14 to 7x7
        {"name": "conv3x3_s2_7", "kind": "conv", "S": 512, "C": 512, "H": 14, "batch": 256, "k": 3, "stride": 2, "n": 4, "m": 8,
         "B": 64, "d": 0.4, "bf16": 1, "ep": 1},
        # the network as it is served: a small batch, where latency and launches count ...
        {"name": "resnet50_b8", "kind": "net", "batch": 8, "plan": 0},
        # ... and a large one
        {"name": "resnet50_b256", "kind": "net", "batch": 256, "plan": 0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """A channel count: mostly multiples of 64 or 16 as networks have them, some odd ones."""
    c = _log_int(rng, lo, hi)
    step = rng.choice((64, 64, 64, 16, 8, 1))
    return max(step, c // step * step) if step > 1 else c


def _topk_fits(S, K, B):
    """Whole-grid block choice takes grids of up to 8192 blocks."""
    return -(-S // B) * -(-K // B) <= 8192


def draw(rng):
    kind = rng.choice(("prune", "model", "gemm", "gemm", "gemm", "gemm", "conv", "conv", "conv", "net"))
    n, m = rng.choice(PATTERNS)
    B = rng.choice((64, 64, 64, 32, 32, 16))
    d = round(rng.uniform(0.2, 0.8), 3)
    if kind == "prune":
        S, K = _channels(rng, 24, 2048), _channels(rng, 64, 4608)
        return {"kind": kind, "S": S, "K": K, "n": n, "m": m, "B": B, "d": d, "sal": rng.choice((0, 1, 2)),
                "topk": int(rng.random() < 0.15 and _topk_fits(S, K, B))}
    if kind == "model":
        return {"kind": kind, "B": rng.choice((32, 64)), "plan": rng.randrange(1, 1 << 20)}
    if kind == "net":
        return {"kind": kind, "batch": 8 * _log_int(rng, 1, 32), "plan": rng.randrange(1, 1 << 20)}
    if kind == "gemm":
        S, K = _channels(rng, 24, 2048), _channels(rng, 64, 4608)
        N = min(_log_int(rng, 49, 401408), (1 << 28) // max(S, K), (1 << (32 if B == 16 else 34)) // (S * K) * 8)
        if rng.random() < 0.75:
            N = max(8, N // 8 * 8)
        topk = int(rng.random() < 0.15 and _topk_fits(S, K, B))
        k8 = int(rng.random() < 0.15 and B != 16 and K % 16 == 0 and S % 8 == 0)
        ep = int(rng.random() < 0.5)
        return {"kind": kind, "S": S, "K": K, "N": N, "n": n, "m": m, "B": B, "d": d, "bf16": int(rng.random() < 0.75), "ep": ep,
                "res": int(ep and rng.random() < 0.5), "k8": k8, "topk": topk}
    k, stride = rng.choice(((1, 1), (1, 2), (3, 1), (3, 1), (3, 1), (3, 2), (5, 1), (7, 2)))
    C = rng.choice((3, 3, 4)) if k == 7 else _channels(rng, 24, 512)
    H = rng.choice((224, 112, 160)) if k == 7 else rng.choice((7, 14, 28, 56, 13, 20, 33))
    batch = _log_int(rng, 1, 256)
    batch = max(1, min(batch, (1 << 27) // (H * H * max(C, 32)), (1 << 34) // (H * H * C * k * k * 64) * 8))
    return {"kind": kind, "S": min(_channels(rng, 24, 1024), 256 if k > 3 else 1024), "C": C, "H": H, "batch": batch, "k": k,
            "stride": stride, "n": n, "m": m, "B": 64 if B == 16 else B, "d": d, "bf16": int(rng.random() < 0.75),
            "ep": int(rng.random() < 0.5)}


# ---- inputs ---------------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _bits(t):
    return t.to(torch.bfloat16).view(torch.int16)


def _weight(g, S, K):
    return _bits(torch.randn((S, K), generator=g, device="cuda") * math.sqrt(2.0 / K))


def _activation(g, shape):
    """ReLU(N(0, 1)), drawn in pieces so that the fp32 values never take more than a fraction of the result."""
    out = torch.empty(shape, dtype=torch.int16, device="cuda")
    flat = out.view(-1)
    for i in range(0, flat.numel(), 1 << 26):
        part = flat[i:i + (1 << 26)]
        part.copy_(_bits(torch.randn(part.numel(), generator=g, device="cuda").clamp_(min=0)))
    return out


def _plan(case):
    """The 53 layers with their drawn patterns and densities; plan 0 is the benchmark's own draw."""
    wl = synth.resnet50(case.get("batch", 1), synth.SEED_BASE + 5 + case["plan"])
    for L in wl.layers:
        L.B = case.get("B", L.B)
    return wl


def _packed(g, S, K, n, m, B, d, topk=0):
    desc = crisp.layer_desc(S, K, n, m, B, d, crisp.SAL_GRAD, crisp.LAYER_TOPK if topk else crisp.ROW_UNIFORM)
    layer = crisp.alloc_layer(desc)
    W, G = _weight(g, S, K), torch.randn((S, K), generator=g, device="cuda")
    crisp.prune_and_pack(layer, W, G)
    layer.ws = None
    return layer


FIELDS = ("nm_mask", "row_ptr", "col_idx", "score", "vals", "idx_words", "flags")


def _model(g, wl):
    """Layers, weights and gradients of the network; the layers' buffers of one kind lie in one allocation."""
    layers, Ws, Gs = [], [], []
    for L in wl.layers:
        layers.append(crisp.alloc_layer(crisp.layer_desc(L.S, L.K, L.n, L.m, L.B, L.density, L.sal_kind)))
        Ws.append(_weight(g, L.S, L.K))
        Gs.append(torch.randn((L.S, L.K), generator=g, device="cuda"))
    arenas = []
    for f in FIELDS:
        sizes = [-(-getattr(layer, f).numel() // 64) * 64 for layer in layers]
        arena = torch.zeros(sum(sizes), dtype=getattr(layers[0], f).dtype, device="cuda")
        at = 0
        for layer, size in zip(layers, sizes):
            setattr(layer, f, arena[at:at + getattr(layer, f).numel()])
            at += size
        arenas.append(arena)
    return layers, Ws, Gs, arenas


def _round8(n):
    return (n + 7) // 8 * 8


def _conv_shape(case):
    return synth.ConvShape(case["C"], case["H"], case["H"], case["batch"], case["k"], case["k"], case["stride"], case["k"] // 2)


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    st = {"case": case}
    if kind == "prune":
        S, K = case["S"], case["K"]
        desc = crisp.layer_desc(S, K, case["n"], case["m"], case["B"], case["d"], case["sal"],
                                crisp.LAYER_TOPK if case["topk"] else crisp.ROW_UNIFORM)
        st["layer"] = crisp.alloc_layer(desc)
        st["W"] = _weight(g, S, K)
        t = torch.randn((S, K), generator=g, device="cuda")
        st["TG"] = None if case["sal"] == crisp.SAL_MAG else t.abs() if case["sal"] == crisp.SAL_GIVEN else t
        st["layer"].nm_mask.zero_()
    elif kind == "model":
        layers, Ws, Gs, arenas = _model(g, _plan(case))
        st.update(layers=layers, Ws=Ws, Gs=Gs, arenas=arenas, batch=crisp.make_batch(layers, Ws, Gs))
    elif kind == "gemm":
        S, K, N = case["S"], case["K"], case["N"]
        st["layer"] = _packed(g, S, K, case["n"], case["m"], case["B"], case["d"], case["topk"])
        ld = st["ld"] = _round8(N)
        k8 = case["k8"]
        st["X"] = _activation(g, (K // 8, ld, 8) if k8 else (K, ld))
        ydt = torch.bfloat16 if case["bf16"] else torch.float32
        st["Y"] = torch.empty((S // 8, ld, 8) if k8 else (S, ld), dtype=ydt, device="cuda")
        st["ep"] = None
        if case["ep"]:
            st["scale"] = torch.rand(S, generator=g, device="cuda") + 0.5
            st["bias"] = torch.randn(S, generator=g, device="cuda") * 0.1
            st["res"] = None
            if case["res"]:
                st["res"] = torch.randn(st["Y"].shape, generator=g, device="cuda").to(ydt)
            st["ep"] = crisp.epilogue(st["scale"], st["bias"], st["res"], ld if case["res"] else 0, True)
    elif kind == "conv":
        cv = st["cv"] = _conv_shape(case)
        st["layer"] = _packed(g, case["S"], cv.K, case["n"], case["m"], case["B"], case["d"])
        ld = st["ld"] = _round8(cv.Ncol)
        st["act"] = _activation(g, (cv.C, cv.batch, cv.H, cv.W))
        st["Y"] = torch.empty((case["S"], ld), dtype=torch.bfloat16 if case["bf16"] else torch.float32, device="cuda")
        nbytes = crisp.conv_plan(st["layer"].desc, cv)[1]
        st["scratch"] = torch.empty(nbytes // 2, dtype=torch.int16, device="cuda") if nbytes else None
        st["ep"] = None
        if case["ep"]:
            st["scale"] = torch.rand(case["S"], generator=g, device="cuda") + 0.5
            st["bias"] = torch.randn(case["S"], generator=g, device="cuda") * 0.1
            st["ep"] = crisp.epilogue(st["scale"], st["bias"], None, 0, True)
    else:
        wl = st["wl"] = _plan(case)
        layers, Ws, Gs, _ = _model(g, wl)
        crisp.crisp_select_pack_batch(*crisp.make_batch(layers, Ws, Gs))
        torch.cuda.synchronize()               # the weights and gradients are let go of below
        for layer in layers:
            layer.ws = None
        st["layers"] = layers
        st["scales"] = resnet.layer_scales(wl, layers)
        st["x"] = _activation(g, (3, case["batch"], 224, 224))
        nbytes = max(crisp.conv_plan(layer.desc, L.conv)[1] for L, layer in zip(wl.layers, layers))
        st["scratch"] = torch.empty(nbytes // 2, dtype=torch.int16, device="cuda") if nbytes else None
    return st


# ---- one pass -------------------------------------------------------------------------------------------------

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "prune":
        crisp.prune_and_pack(st["layer"], st["W"], st["TG"])
        return [getattr(st["layer"], f) for f in FIELDS]
    if kind == "model":
        crisp.crisp_select_pack_batch(*st["batch"])
        return st["arenas"]
    if kind == "gemm":
        layer = st["layer"]
        ydt = crisp.Y_BF16 if case["bf16"] else crisp.Y_F32
        xl = crisp.X_K8 if case["k8"] else crisp.X_KN
        if st["ep"] is None:
            crisp.crisp_spmm(layer.desc, layer.row_ptr, layer.col_idx, layer.vals, layer.idx_words, st["X"], case["N"], st["ld"],
                             st["Y"], st["ld"], ydt, x_layout=xl)
        else:
            crisp.crisp_spmm_ep(layer.desc, layer.row_ptr, layer.col_idx, layer.vals, layer.idx_words, st["X"], case["N"],
                                st["ld"], st["Y"], st["ld"], ydt, st["ep"], x_layout=xl)
        return st["Y"] if st["ld"] == case["N"] else st["Y"][:, :case["N"]]
    if kind == "conv":
        crisp.conv_forward(st["layer"], st["cv"], st["act"], st["Y"], st["ld"], crisp.Y_BF16 if case["bf16"] else crisp.Y_F32,
                           st["scratch"], st["ep"])
        return st["Y"] if st["ld"] == st["cv"].Ncol else st["Y"][:, :st["cv"].Ncol]
    return resnet.forward(st["wl"], st["layers"], st["x"], st["scales"], st["scratch"]).view(torch.bfloat16)


# ---- what a pass cannot do without ----------------------------------------------------------------------------

def _packed_bytes(sz, B):
    return sz.vals_elems * 2 + sz.idx_words * 4 + sz.col_idx_elems * 4 + sz.row_ptr_elems * 4


def _used(Kb, Sb, k_row):
    """Expected share of the block columns that at least one block-row keeps."""
    return 1.0 - (1.0 - k_row / Kb) ** Sb


def _prune_bytes(S, K, n, m, B, d, sal):
    sz = crisp.crisp_pack_sizes(crisp.layer_desc(S, K, n, m, B, d))
    return S * K * (2 + (0 if sal == 2 else 4)) + sz.mask_words * 4 + sz.score_elems * 8 + _packed_bytes(sz, B)


def _product(S, K, N, n, m, B, d, x_elems, y_bytes, res, taps=1):
    sz = crisp.crisp_pack_sizes(crisp.layer_desc(S, K, n, m, B, d))
    share = _used(sz.Kb, sz.Sb, sz.k_row) if taps == 1 else 1.0    # several taps: practically every channel is used by one
    return {"bytes": int(x_elems * 2 * share + S * N * y_bytes * (2 if res else 1) + _packed_bytes(sz, B)),
            "flops": int(2 * S * N * K * (sz.k_row / sz.Kb) * n / m)}


def work(case):
    kind = case["kind"]
    if kind == "prune":
        return {"bytes": _prune_bytes(case["S"], case["K"], case["n"], case["m"], case["B"], case["d"], case["sal"]), "flops": 0}
    if kind == "model":
        return {"bytes": sum(_prune_bytes(L.S, L.K, L.n, L.m, L.B, L.density, L.sal_kind) for L in _plan(case).layers), "flops": 0}
    if kind == "gemm":
        return _product(case["S"], case["K"], case["N"], case["n"], case["m"], case["B"], case["d"], case["K"] * case["N"],
                        2 if case["bf16"] else 4, case["res"])
    if kind == "conv":
        cv = _conv_shape(case)
        touched = cv.Ho * cv.Wo if cv.kh == 1 else cv.H * cv.W      # a strided 1x1 filter skips input positions
        return _product(case["S"], cv.K, cv.Ncol, case["n"], case["m"], case["B"], case["d"], cv.C * cv.batch * touched,
                        2 if case["bf16"] else 4, 0, cv.kh * cv.kw)
    total = {"bytes": 0, "flops": 0}
    for L in _plan(case).layers:
        cv = L.conv
        touched = cv.Ho * cv.Wo if cv.kh == 1 else cv.H * cv.W
        w = _product(L.S, L.K, L.Ncol, L.n, L.m, L.B, L.density, cv.C * cv.batch * touched, 2, L.name.endswith(".c"), cv.kh * cv.kw)
        total["bytes"] += w["bytes"]
        total["flops"] += w["flops"]
    total["bytes"] += 64 * case["batch"] * (112 * 112 + 56 * 56) * 2      # the max-pool between the first two stages
    return total


def tolerance(case):
    kind = case["kind"]
    if kind in ("prune", "model"):
        return "exact"                       # total orders and a fixed summation order: every byte is determined
    # about four times the distance from the same path in 64 bits: fp32 results differ by 2e-8 ... 7e-8 (order of the
    # sums; the products are exact), bf16 results by the one rounding at the end (1.66e-3), the network by the
    # roundings of 53 layers (7e-3 ... 9e-3)
    if kind == "net":
        return {"rel": 3.6e-2}
    return {"rel": 6.6e-3} if case["bf16"] else {"rel": 4e-7}
