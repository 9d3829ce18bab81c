"""The kernels in which four or eight waves split a tile's block list: a strided convolution with long block lists, in
every split, against the oracle and bit for bit against the explicit lowering in the same launch shape, with the input
at another address in every launch."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_14272_amd import crisp, synth

from gpu_util import check_product, dev, run_select_pack, run_spmm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,B", [(2, 4, 64), (3, 4, 64), (1, 8, 32)])
@pytest.mark.parametrize("geom", [(128, 22, 41, 4, 7, 2, 3), (64, 9, 20, 2, 3, 2, 1)])
def test_split_repeats_itself(n, m, B, geom):
    C_, H, W_, b, k, stride, pad = geom
    cv = synth.ConvShape(C_, H, W_, b, k, k, stride, pad)
    L = synth.LayerSpec("split", 64, cv.K, cv.Ncol, n, m, B, 0.5, synth.SAL_MAG, 0.05, conv=cv)
    rng = np.random.default_rng(n * 100 + m + C_)
    W, act = synth.draw_weight(rng, L), synth.draw_relu_normal(rng, (C_, b, H, W_))
    sel = oracle.select(W, None, n, m, B, 0.5, synth.SAL_MAG, L.select_mode)
    X = oracle.im2col(act, k, k, stride, pad)
    Yref, Aref = oracle.gemm_masked(W, sel.mask, X)
    layer, _ = run_select_pack(L, W, None)
    conv, Ncol, ld = crisp.conv_desc_of(cv), cv.Ncol, (cv.Ncol + 7) // 8 * 8
    dact = dev(act).reshape(-1)
    pool = torch.empty(8 * (dact.numel() + 64), dtype=torch.int16, device="cuda")
    Xp = np.zeros((cv.K, ld), dtype=np.uint16)
    Xp[:, :Ncol] = X
    dX = dev(Xp)
    for shape, split in ((2, 2), (3, 3), (9, 2), (10, 3)):
        explicit = run_spmm(layer, dX, Ncol, ld, crisp.Y_F32, L.S, shape=shape)
        check_product(explicit, Yref, Aref, crisp.Y_F32, "explicit, shape %d" % shape)
        for rep in range(8):
            at = rep * ((dact.numel() + 64) // 8 * 8)
            moved = pool[at:at + dact.numel()]
            moved.copy_(dact)
            Y = torch.full((L.S, ld), float("nan"), dtype=torch.float32, device="cuda")
            code = crisp.crisp_conv_spmm_forced(layer.desc, conv, layer.row_ptr, layer.col_idx, layer.vals, layer.idx_words,
                                                moved, Y, ld, crisp.Y_F32, None, shape)
            torch.cuda.synchronize()
            fields = crisp.kernel_code_fields(code)
            assert (fields["family"], fields["shape"], fields["conv_mode"]) == ("reg", split, 2)
            got = Y.cpu().numpy().astype(np.float64)[:, :Ncol]
            assert (got == explicit).all(), "shape %d, launch %d: %d outputs differ" % (shape, rep, int((got != explicit).sum()))


@pytest.mark.parametrize("n,m", [(3, 4), (4, 4), (4, 8), (8, 8), (2, 4), (1, 8)])
@pytest.mark.parametrize("B", [32, 64])
def test_split_by_eight_is_never_the_librarys_choice(n, m, B):
    """Few tiles and long block lists, where it used to be: plain X and a convolution."""
    L = synth.LayerSpec("choice", 128, 1152, 196, n, m, B, 1.0, synth.SAL_MAG, 0.05)
    rng = np.random.default_rng(n * 10 + m)
    W = synth.draw_weight(rng, L)
    layer, _ = run_select_pack(L, W, None)
    X = torch.zeros((1152, 200), dtype=torch.int16, device="cuda")
    Y = torch.empty((128, 200), dtype=torch.float32, device="cuda")
    args = (layer.row_ptr, layer.col_idx, layer.vals, layer.idx_words, X)
    plain = crisp.crisp_spmm_forced(layer.desc, *args, 196, 200, Y, 200, crisp.Y_F32, None, crisp.SHAPE_AUTO)
    conv = crisp.crisp_conv_spmm_forced(layer.desc, crisp.ConvDesc(128, 14, 14, 1, 3, 3, 1, 1, crisp.ACT_CBHW, crisp.X_KN),
                                        *args, Y, 200, crisp.Y_F32, None, crisp.SHAPE_AUTO)
    torch.cuda.synchronize()
    for code in (plain, conv):
        fields = crisp.kernel_code_fields(code)
        assert fields["family"] == "reg" and fields["shape"] == 2, fields


# C, S, H, batch, k, stride, density, n, m: the kernel that stages the input where it is the faster one (after #, us of
# the register kernels / staged), the register kernels' split by four where few workgroups would leave it idle
@pytest.mark.parametrize("case,family", [
    ((128, 768, 28, 8, 5, 1, 1.0, 2, 4), "conv_lds"),       # 102 / 43
    ((128, 256, 8, 16, 7, 2, 0.8, 2, 4), "conv_lds"),       # 76 / 46
    ((64, 256, 8, 8, 5, 2, 1.0, 2, 4), "conv_lds"),         # 27 / 18
    ((256, 192, 8, 32, 5, 4, 1.0, 8, 8), "conv_lds"),       # 195 / 75
    ((384, 256, 16, 64, 3, 2, 1.0, 1, 4), "conv_lds"),      # 57 / 43: planes of 2^14 elements
    ((256, 256, 14, 8, 3, 1, 0.6, 2, 4), "reg"),            # 10 / 24
    ((128, 128, 56, 8, 3, 2, 0.6, 2, 4), "reg"),            # 12 / 20
    ((512, 512, 8, 8, 3, 1, 0.6, 3, 4), "reg"),             # 17 / 66
], ids=str)
def test_choice_for_few_workgroups(case, family):
    C_, S, H, b, k, stride, dens, n, m = case
    cv = synth.ConvShape(C_, H, H, b, k, k, stride, k // 2)
    layer = crisp.alloc_layer(crisp.layer_desc(S, cv.K, n, m, 64, dens, crisp.SAL_MAG))
    g = torch.Generator(device="cuda").manual_seed(C_)
    W = (torch.randn((S, cv.K), generator=g, device="cuda") * 0.05).to(torch.bfloat16).view(torch.int16)
    crisp.prune_and_pack(layer, W, None)
    act = torch.randn((C_, b, H, H), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16)
    ld = (cv.Ncol + 7) // 8 * 8
    out = []
    for shape in (crisp.SHAPE_AUTO, 12, 2):
        Y = torch.full((S, ld), float("nan"), dtype=torch.float32, device="cuda")
        code = crisp.crisp_conv_spmm_forced(layer.desc, crisp.conv_desc_of(cv), layer.row_ptr, layer.col_idx, layer.vals,
                                            layer.idx_words, act, Y, ld, crisp.Y_F32, None, shape)
        torch.cuda.synchronize()
        out.append((crisp.kernel_code_fields(code)["family"], Y[:, :cv.Ncol]))
    assert out[0][0] == family
    for _, y in out[1:]:
        # the same products in another order: relative 2-norm as of the fp32 tripwire of the parity tests
        assert float((y - out[0][1]).norm() / y.norm()) <= 1e-5
