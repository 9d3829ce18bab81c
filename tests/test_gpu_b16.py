"""16 x 16 blocks, two kept blocks per matrix-core instruction: a wave per block-row and a list split over four waves,
odd and even list lengths, K and column counts that divide nothing, uneven rows, tails, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_14272_amd import crisp, synth

from gpu_util import check_bf16_is_rounded_f32, check_product, dev, run_select_pack

pytestmark = pytest.mark.gpu

PATTERNS = [(1, 4), (2, 4), (3, 4), (4, 4), (1, 8), (2, 8), (3, 8), (4, 8), (8, 8)]


def _run(layer, X, N, ld, S, yd, ep=None):
    Y = torch.full((S + 1, ld), float("nan"), dtype=torch.float32 if yd == crisp.Y_F32 else torch.bfloat16, device="cuda")
    code = crisp.crisp_spmm_forced(layer.desc, layer.row_ptr, layer.col_idx, layer.vals, layer.idx_words, X, N, ld, Y, ld, yd, ep)
    torch.cuda.synchronize()
    Yh = Y.float().cpu().numpy().astype(np.float64)
    assert np.isnan(Yh[:S, N:]).all() and np.isnan(Yh[S]).all(), "guard band written"
    f = crisp.kernel_code_fields(code)
    assert f["family"] == "b16"
    return Yh[:S, :N], f["shape"]


# S, K, N, density, whole-grid choice, kernel (1 a wave per block-row, 2 split list)
@pytest.mark.parametrize("case", [
    (64, 64, 128, 0.3, 0, 1),          # one block per row: the pair's second block is absent
    (100, 96, 131, 0.5, 0, 1),         # three blocks, ragged rows and columns
    (48, 200, 77, 1.0, 0, 2),          # thirteen blocks over four waves, K no multiple of 16
    (16, 1030, 200, 0.5, 0, 2),        # K = 6 mod 16, one block-row
    (130, 512, 9, 0.9, 0, 2),
    (96, 320, 264, 0.35, 1, 1),        # uneven and empty rows
], ids=lambda c: "S%d_K%d_N%d" % c[:3])
def test_pairs_of_blocks(case):
    S, K, N, dens, topk, kernel = case
    for n, m in PATTERNS:
        L = synth.LayerSpec("b16", S, K, N, n, m, 16, dens, synth.SAL_MAG, 0.05, select_mode=synth.LAYER_TOPK if topk else synth.ROW_UNIFORM)
        rng = np.random.default_rng(S + K + n)
        W = synth.draw_weight(rng, L)
        X = synth.draw_relu_normal(rng, (K, N))
        sel = oracle.select(W, None, n, m, 16, dens, synth.SAL_MAG, L.select_mode)
        layer, _ = run_select_pack(L, W, None)
        Yref, Aref = oracle.gemm_masked(W, sel.mask, X)
        ld = (N + 7) // 8 * 8 + 8
        Xp = np.zeros((K, ld), dtype=np.uint16)
        Xp[:, :N] = X
        dX = dev(Xp)
        f32, shape = _run(layer, dX, N, ld, S, crisp.Y_F32)
        assert shape == (0 if (n, m) == (3, 8) else kernel)
        check_product(f32, Yref, Aref, crisp.Y_F32, "%s %d:%d" % (case, n, m))
        b16, _ = _run(layer, dX, N, ld, S, crisp.Y_BF16)
        check_bf16_is_rounded_f32(b16, f32, "%s %d:%d" % (case, n, m))
        g = torch.Generator(device="cuda").manual_seed(1)
        scale, bias, res = torch.rand(S, generator=g, device="cuda"), torch.randn(S, generator=g, device="cuda"), torch.randn((S, ld), generator=g, device="cuda")
        out, _ = _run(layer, dX, N, ld, S, crisp.Y_F32, crisp.epilogue(scale, bias, res, ld, True))
        want = torch.relu(torch.from_numpy(f32).cuda().float() * scale[:, None] + bias[:, None] + res[:, :N])
        assert (torch.from_numpy(out).cuda().float() == want).all()


@pytest.mark.parametrize("K", [48, 44])
def test_infinite_activation_outside_the_kept_blocks_stays_outside(K):
    """Rows of X that no kept block reads, and K-rows past the end, take no part: with an odd list the second half of the
    last pair is zero in both operands."""
    S, N, n, m = 32, 40, 2, 4
    L = synth.LayerSpec("inf", S, K, N, n, m, 16, 0.34, synth.SAL_MAG, 0.05)
    rng = np.random.default_rng(K)
    W = synth.draw_weight(rng, L)
    X = synth.draw_relu_normal(rng, (K, N))
    sel = oracle.select(W, None, n, m, 16, 0.34, synth.SAL_MAG, L.select_mode)
    kept = {int(b) for b in sel.col_idx}
    layer, _ = run_select_pack(L, W, None)
    Yref, Aref = oracle.gemm_masked(W, sel.mask, X)
    for b in range(-(-K // 16)):
        if b not in kept:
            X[b * 16:(b + 1) * 16] = 0x7F80
    out, _ = _run(layer, dev(np.ascontiguousarray(X)), N, N, S, crisp.Y_F32)
    check_product(out, Yref, Aref, crisp.Y_F32, "infinite rows")


@pytest.mark.parametrize("S,K,N,dens", [(100, 96, 131, 0.5), (48, 200, 77, 1.0), (64, 64, 128, 0.3), (21, 48, 3, 1.0)])
@pytest.mark.parametrize("parts", ["scale", "bias", "residual", "relu", "all"])
def test_tail_of_rows_that_end_inside_a_lane(S, K, N, dens, parts):
    """Every part of the layer tail alone and all together, both output types: the same fp32 steps in their order, and nothing
    taken from the residual's columns past the last one (NaN there)."""
    g = torch.Generator(device="cuda").manual_seed(S + N)
    layer = crisp.alloc_layer(crisp.layer_desc(S, K, 2, 8, 16, dens, crisp.SAL_MAG))
    crisp.prune_and_pack(layer, torch.randn((S, K), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16), None)
    ld = (N + 7) // 8 * 8
    X = torch.randn((K, ld), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16)
    plain = torch.from_numpy(_run(layer, X, N, ld, S, crisp.Y_F32)[0]).cuda().float()
    scale, bias = torch.rand(S, generator=g, device="cuda") + 0.5, torch.randn(S, generator=g, device="cuda")
    for yd, dtype in ((crisp.Y_F32, torch.float32), (crisp.Y_BF16, torch.bfloat16)):
        res = torch.full((S, ld + 8), float("nan"), dtype=dtype, device="cuda")
        res[:, :N] = torch.randn((S, N), generator=g, device="cuda").to(dtype)
        use = {p: parts in (p, "all") for p in ("scale", "bias", "residual", "relu")}
        want = plain * scale[:, None] if use["scale"] else plain.clone()
        want = want + bias[:, None] if use["bias"] else want
        want = want + res[:, :N].float() if use["residual"] else want
        want = (torch.relu(want) if use["relu"] else want).to(dtype).double()
        ep = crisp.epilogue(scale if use["scale"] else None, bias if use["bias"] else None, res if use["residual"] else None,
                            ld + 8 if use["residual"] else 0, use["relu"])
        out, _ = _run(layer, X, N, ld, S, yd, ep)
        assert (torch.from_numpy(out).cuda() == want).all(), (parts, dtype)
