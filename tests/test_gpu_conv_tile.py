"""The convolution kernel that stages a window of input positions (forced shape 19): images narrower and wider than a
tile, odd widths, several images per tile, parts of an image, strides that skip rows, ragged block-rows, both block
sizes, several channel chunks, uneven and empty block-rows, every pattern -- against the oracle; and the whole
convolution's choice between it and a materialised X."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_14272_amd import crisp, synth

from gpu_util import check_bf16_is_rounded_f32, check_product, dev, run_select_pack

pytestmark = pytest.mark.gpu

PATTERNS = [(1, 4), (2, 4), (3, 4), (4, 4), (1, 8), (2, 8), (4, 8), (8, 8)]


def _layer(case, n, m, select_mode=synth.ROW_UNIFORM):
    S, C_, H, W_, b, kh, kw, stride, pad, B, dens = case
    cv = synth.ConvShape(C_, H, W_, b, kh, kw, stride, pad)
    L = synth.LayerSpec("tile", S, cv.K, cv.Ncol, n, m, B, dens, synth.SAL_MAG, 0.05, conv=cv, select_mode=select_mode)
    rng = np.random.default_rng(S * 31 + C_ + H * 7 + n)
    W = synth.draw_weight(rng, L)
    if select_mode == synth.LAYER_TOPK:          # some block-rows long, some empty
        Wf = synth.bf16_bits_to_f32(W).reshape(S, cv.K)
        Wf[:B] *= 8.0
        Wf[2 * B:3 * B] *= 0.01
        W = synth.f32_to_bf16_bits(Wf.astype(np.float32))
    act = synth.draw_relu_normal(rng, (C_, b, H, W_))
    act[:, :, 0, 0] = synth.f32_to_bf16_bits(np.full((C_, b), 3.0, dtype=np.float32))    # make the borders matter
    act[:, :, -1, -1] = synth.f32_to_bf16_bits(np.full((C_, b), 5.0, dtype=np.float32))
    sel = oracle.select(W, None, n, m, B, dens, synth.SAL_MAG, select_mode)
    layer, _ = run_select_pack(L, W, None)
    Yref, Aref = oracle.gemm_masked(W, sel.mask, oracle.im2col(act, kh, kw, stride, pad))
    return cv, layer, act, Yref, Aref, np.diff(sel.row_ptr)


def _run(cv, layer, act, S, yd, ep=None, guard=8):
    ld = (cv.Ncol + 7) // 8 * 8 + guard
    Y = torch.full((S + 1, ld), float("nan"), dtype=torch.float32 if yd == crisp.Y_F32 else torch.bfloat16, device="cuda")
    code = crisp.crisp_conv_spmm_forced(layer.desc, crisp.conv_desc_of(cv), layer.row_ptr, layer.col_idx, layer.vals, layer.idx_words,
                                        act, Y, ld, yd, ep, 19)
    torch.cuda.synchronize()
    f = crisp.kernel_code_fields(code)
    assert f["family"] == "conv_lds" and f["shape"] in (1, 2), f
    Yh = Y.float().cpu().numpy().astype(np.float64)
    assert np.isnan(Yh[:S, cv.Ncol:]).all() and np.isnan(Yh[S]).all(), "guard band written"
    return Yh[:S, :cv.Ncol]


# S, C, H, W, batch, kh, kw, stride, pad, B, density
@pytest.mark.parametrize("case", [
    (64, 64, 7, 7, 2, 3, 3, 1, 1, 64, 0.5),        # two small images in one tile
    (512, 512, 7, 7, 6, 3, 3, 1, 1, 64, 0.3),      # many block-rows, every channel in one chunk
    (256, 256, 14, 14, 3, 3, 3, 1, 1, 64, 0.6),
    (130, 128, 28, 28, 2, 3, 3, 1, 1, 64, 0.5),    # parts of an image, last block-row of two rows
    (64, 64, 56, 56, 1, 3, 3, 1, 1, 64, 0.7),
    (200, 512, 14, 14, 4, 3, 3, 2, 1, 64, 0.4),    # several chunks
    (96, 128, 33, 33, 2, 3, 3, 2, 1, 64, 0.5),     # odd widths, odd output positions per image
    (320, 64, 13, 13, 4, 5, 5, 1, 2, 64, 0.3),
    (250, 64, 20, 9, 2, 3, 5, 3, 0, 64, 0.5),      # uneven filter, stride 3, no padding
    (40, 32, 13, 13, 2, 3, 3, 1, 1, 32, 0.5),      # 32 x 32 blocks
    (352, 160, 14, 14, 4, 3, 3, 2, 1, 32, 0.4),
    (64, 64, 5, 4, 2, 3, 3, 1, 2, 64, 1.0),        # narrowest image, padding of two
    (72, 24, 14, 14, 2, 3, 3, 1, 1, 64, 0.5),      # block columns of several taps, K no multiple of 16
    (64, 8, 12, 12, 2, 5, 5, 1, 2, 64, 1.0),
    (100, 200, 13, 13, 2, 3, 3, 1, 1, 64, 0.4),
    (96, 40, 20, 20, 2, 3, 3, 2, 1, 32, 0.6),
    (300, 272, 28, 28, 2, 3, 3, 2, 1, 64, 0.2),    # ... over several chunks
], ids=lambda c: "S%d_C%d_%dx%d_k%ds%d_B%d" % (c[0], c[1], c[2], c[3], c[5], c[7], c[9]))
def test_window_kernel_against_the_oracle(case):
    for n, m in PATTERNS if case[0] * case[1] <= 20000 else ((2, 8), (4, 8)):
        cv, layer, act, Yref, Aref, _ = _layer(case, n, m)
        dact = dev(act)
        f32 = _run(cv, layer, dact, case[0], crisp.Y_F32)
        check_product(f32, Yref, Aref, crisp.Y_F32, "%s %d:%d" % (case, n, m))
        check_bf16_is_rounded_f32(_run(cv, layer, dact, case[0], crisp.Y_BF16), f32, "%s %d:%d" % (case, n, m))


@pytest.mark.parametrize("n,m", [(2, 4), (4, 8)])
def test_window_kernel_with_uneven_and_empty_block_rows(n, m):
    case = (448, 128, 14, 14, 2, 3, 3, 1, 1, 64, 0.2)
    cv, layer, act, Yref, Aref, counts = _layer(case, n, m, synth.LAYER_TOPK)
    assert counts.min() == 0 and counts.max() > 4
    check_product(_run(cv, layer, dev(act), case[0], crisp.Y_F32), Yref, Aref, crisp.Y_F32, "uneven")


def test_window_kernel_tail():
    """Scale, bias, residual and ReLU, as in every other kernel: fp32 steps in their order, one rounding each."""
    case = (200, 64, 28, 28, 1, 3, 3, 1, 1, 64, 0.5)
    cv, layer, act, Yref, Aref, _ = _layer(case, 2, 8)
    S, dact, ld = case[0], dev(act), (cv.Ncol + 7) // 8 * 8
    plain = torch.from_numpy(_run(cv, layer, dact, S, crisp.Y_F32).astype(np.float32)).cuda()
    g = torch.Generator(device="cuda").manual_seed(3)
    scale, bias = torch.rand(S, generator=g, device="cuda") + 0.5, torch.randn(S, generator=g, device="cuda")
    res = torch.randn((S, ld), generator=g, device="cuda")
    out = _run(cv, layer, dact, S, crisp.Y_F32, crisp.epilogue(scale, bias, res, ld, True))
    want = torch.relu(plain * scale[:, None] + bias[:, None] + res[:, :cv.Ncol])
    assert (torch.from_numpy(out).cuda().float() == want).all()
    res16 = res.to(torch.bfloat16)
    out = _run(cv, layer, dact, S, crisp.Y_BF16, crisp.epilogue(scale, bias, res16, ld, True))
    want = torch.relu(plain * scale[:, None] + bias[:, None] + res16[:, :cv.Ncol].float()).to(torch.bfloat16)
    assert (torch.from_numpy(out).cuda() == want.double()).all()


def test_planned_lowering_gives_way_to_the_window_kernel():
    """A strided 3x3 layer that is planned through a materialised X: run fused where there are columns enough, with the plan
    and its scratch as they were; through X for few columns and for output rows beyond the fused kernels' stride."""
    S, n, m = 256, 4, 8
    for b, d, ldy_extra, expect in ((192, 0.45, 0, "fused"), (2, 0.8, 0, "im2col"), (192, 0.45, (1 << 23) + 8, "im2col")):
        case = (S, 128, 14, 14, b, 3, 3, 2, 1, 64, d)
        cv, layer, act, Yref, Aref, _ = _layer(case, n, m)
        planned, nbytes = crisp.conv_plan(layer.desc, cv)
        assert planned == "im2col" and nbytes == cv.K * ((cv.Ncol + 7) // 8 * 8) * 2
        ldy = ldy_extra or (cv.Ncol + 7) // 8 * 8
        Y = torch.empty((S, ldy), dtype=torch.float32, device="cuda")
        dact = dev(act)
        with pytest.raises(ValueError):
            crisp.conv_forward(layer, cv, dact, Y, ldy, crisp.Y_F32, None)
        X = torch.empty(nbytes // 2, dtype=torch.int16, device="cuda")
        assert crisp.conv_forward(layer, cv, dact, Y, ldy, crisp.Y_F32, X) == expect
        torch.cuda.synchronize()
        check_product(Y[:, :cv.Ncol].cpu().numpy().astype(np.float64), Yref, Aref, crisp.Y_F32, "batch %d" % b)
        del Y


@pytest.mark.parametrize("case,n,m", [
    ((96, 128, 13, 13, 45, 3, 3, 1, 1, 64, 0.5), 1, 4),
    ((64, 72, 33, 33, 13, 3, 3, 1, 1, 64, 0.6), 4, 8),
    ((40, 64, 7, 7, 301, 5, 5, 1, 2, 32, 0.5), 2, 8),
], ids=str)
def test_odd_number_of_columns(case, n, m):
    """Planned through a materialised X, run from the window: the last lane stores one column, with and without a tail."""
    cv, layer, act, Yref, Aref, _ = _layer(case, n, m)
    S, N = case[0], cv.Ncol
    assert N % 2 == 1 and crisp.conv_plan(layer.desc, cv)[0] == "im2col"
    ld, dact = (N + 7) // 8 * 8, dev(act)
    X = torch.empty(crisp.conv_plan(layer.desc, cv)[1] // 2, dtype=torch.int16, device="cuda")

    def run(yd, ep=None):
        Y = torch.full((S + 1, ld), float("nan"), dtype=torch.float32 if yd == crisp.Y_F32 else torch.bfloat16, device="cuda")
        assert crisp.conv_forward(layer, cv, dact, Y, ld, yd, X, ep) == "fused"
        torch.cuda.synchronize()
        Yh = Y.float().cpu().numpy().astype(np.float64)
        assert np.isnan(Yh[:S, N:]).all() and np.isnan(Yh[S]).all(), "guard band written"
        return Yh[:S, :N]

    f32 = run(crisp.Y_F32)
    check_product(f32, Yref, Aref, crisp.Y_F32, str(case))
    check_bf16_is_rounded_f32(run(crisp.Y_BF16), f32, str(case))
    g = torch.Generator(device="cuda").manual_seed(5)
    scale, bias, res = torch.rand(S, generator=g, device="cuda"), torch.randn(S, generator=g, device="cuda"), torch.randn((S, ld), generator=g, device="cuda")
    want = torch.relu(torch.from_numpy(f32).cuda().float() * scale[:, None] + bias[:, None] + res[:, :N])
    assert (torch.from_numpy(run(crisp.Y_F32, crisp.epilogue(scale, bias, res, ld, True))).cuda().float() == want).all()


@pytest.mark.parametrize("case,n,m,expect", [
    ((320, 704, 13, 13, 24, 1, 1, 2, 0, 64, 0.3), 2, 4, "fused"),      # pairs located one by one
    ((1090, 512, 28, 28, 3, 1, 1, 2, 0, 64, 0.5), 4, 8, "fused"),      # pairs from one 8-byte piece, a remainder of rows
    ((320, 64, 27, 27, 2, 3, 3, 2, 1, 64, 0.5), 3, 4, "fused"),        # several taps, a short list
    ((96, 36, 14, 14, 4, 1, 1, 2, 0, 32, 0.5), 1, 8, "fused"),         # channels that are no multiple of the block edge
    ((320, 64, 27, 27, 2, 3, 3, 2, 1, 32, 0.7), 3, 4, "im2col"),       # several taps, a long list
    ((592, 896, 33, 33, 16, 1, 1, 2, 0, 32, 0.63), 3, 4, "im2col"),    # much to locate
], ids=str)
def test_planned_lowering_gives_way_to_the_register_kernels(case, n, m, expect):
    """Small strided convolutions planned through a materialised X: one launch where the register kernels take less, with the
    same results as X and the product give, epilogue included, and the same refusals."""
    cv, layer, act, Yref, Aref, _ = _layer(case, n, m)
    S, N = case[0], cv.Ncol
    planned, nbytes = crisp.conv_plan(layer.desc, cv)
    assert planned == "im2col" and nbytes == cv.K * ((N + 7) // 8 * 8) * 2
    ld, dact = (N + 7) // 8 * 8, dev(act)
    X = torch.empty(nbytes // 2, dtype=torch.int16, device="cuda")
    Y = torch.full((S + 1, ld), float("nan"), dtype=torch.float32, device="cuda")
    with pytest.raises(ValueError):
        crisp.conv_forward(layer, cv, dact, Y, ld, crisp.Y_F32, None)
    assert crisp.conv_forward(layer, cv, dact, Y, ld, crisp.Y_F32, X) == expect
    torch.cuda.synchronize()
    assert bool(torch.isnan(Y[:S, N:]).all()) and bool(torch.isnan(Y[S]).all())
    plain = Y[:S, :N].clone()
    check_product(plain.cpu().numpy().astype(np.float64), Yref, Aref, crisp.Y_F32, str(case))
    g = torch.Generator(device="cuda").manual_seed(5)
    scale, bias, res = torch.rand(S, generator=g, device="cuda"), torch.randn(S, generator=g, device="cuda"), torch.randn((S, ld), generator=g, device="cuda")
    assert crisp.conv_forward(layer, cv, dact, Y, ld, crisp.Y_F32, X, crisp.epilogue(scale, bias, res, ld, True)) == expect
    assert (Y[:S, :N] == torch.relu(plain * scale[:, None] + bias[:, None] + res[:, :N])).all()
