"""Fused lowering where the first or last element of a channel plane is all that a lane's two columns have inside the
image: against the oracle's lowering and masked product.  The input lies between guard bands of NaN."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_14272_amd import crisp, synth

from gpu_util import check_product, dev, run_select_pack

pytestmark = pytest.mark.gpu

# C, H, W, batch, kh, kw, stride, pad
GEOMS = [(64, 4, 3, 2, 5, 5, 1, 2), (64, 3, 3, 4, 7, 7, 1, 3), (128, 2, 3, 2, 5, 5, 1, 2),
         # padding of more than (k - 1) / 2: rows and columns of the output that see no input at all
         (64, 6, 8, 2, 3, 3, 1, 2), (64, 5, 4, 2, 1, 1, 1, 2), (64, 6, 9, 2, 3, 1, 2, 3), (64, 7, 6, 2, 7, 1, 2, 3),
         (128, 3, 6, 2, 1, 7, 1, 3)]


@pytest.mark.parametrize("geom", GEOMS, ids=lambda g: "C%d_%dx%d_b%d_k%dx%d_s%d_p%d" % g)
@pytest.mark.parametrize("n,m,B", [(2, 4, 64), (3, 4, 32)])
def test_borders(geom, n, m, B):
    C_, H, W_, b, kh, kw, stride, pad = geom
    cv = synth.ConvShape(C_, H, W_, b, kh, kw, stride, pad)
    L = synth.LayerSpec("border", 64, cv.K, cv.Ncol, n, m, B, 1.0, synth.SAL_MAG, 0.05, conv=cv)
    rng = np.random.default_rng(C_ + H)
    W = synth.draw_weight(rng, L)
    act = synth.f32_to_bf16_bits(rng.standard_normal((C_, b, H, W_)).astype(np.float32))
    sel = oracle.select(W, None, n, m, B, 1.0, synth.SAL_MAG, L.select_mode)
    Yref, Aref = oracle.gemm_masked(W, sel.mask, oracle.im2col(act, kh, kw, stride, pad))
    layer, _ = run_select_pack(L, W, None)
    guard = 4096
    around = torch.full((act.size + 2 * guard,), 0x7FC0, dtype=torch.int16, device="cuda")
    dact = around[guard:guard + act.size]
    dact.copy_(dev(act).reshape(-1))
    ld = (cv.Ncol + 7) // 8 * 8
    for shape in (crisp.SHAPE_AUTO, 1, 2, 8, 9):
        Y = torch.full((L.S, ld), float("nan"), dtype=torch.float32, device="cuda")
        code = crisp.crisp_conv_spmm_forced(layer.desc, crisp.conv_desc_of(cv), layer.row_ptr, layer.col_idx, layer.vals,
                                            layer.idx_words, dact, Y, ld, crisp.Y_F32, None, shape)
        torch.cuda.synchronize()
        if shape != crisp.SHAPE_AUTO:
            assert crisp.kernel_code_fields(code)["family"] == "reg"
        check_product(Y.cpu().numpy().astype(np.float64)[:, :cv.Ncol], Yref, Aref, crisp.Y_F32, "shape %d" % shape)
