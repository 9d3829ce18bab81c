"""The residual requested ahead across block-rows (X-resident kernels, bf16 output): against the batch-wise tail of the
fp32 output of the same kernel, whose rounding the bf16 output has to be bit for bit."""
import pytest
import torch

from paper_2311_14272_amd import crisp

pytestmark = pytest.mark.gpu


def _layer(g, S, K, n, m, d):
    layer = crisp.alloc_layer(crisp.layer_desc(S, K, n, m, 64, d, crisp.SAL_MAG))
    W = (torch.randn((S, K), generator=g, device="cuda") * 0.1).to(torch.bfloat16).view(torch.int16)
    crisp.prune_and_pack(layer, W, None)
    return layer


# shape 13: K <= 64 (ring of a whole block-row), shape 18: two to eight block columns (ring of half a one); S with a
# partial last block-row, fewer block-rows than waves, and several groups of block-rows; ragged strips
@pytest.mark.parametrize("shape,K", [(13, 64), (13, 48), (18, 128), (18, 464)])
@pytest.mark.parametrize("S,N", [(64, 68), (100, 516), (203, 260), (1000, 1028), (2304, 132)])
@pytest.mark.parametrize("n,m", [(2, 4), (1, 8), (4, 8), (3, 4)])
@pytest.mark.parametrize("scale,bias,relu", [(1, 1, 1), (0, 0, 0), (1, 0, 0), (0, 1, 1)])
def test_bf16_is_the_rounding_of_fp32(shape, K, S, N, n, m, scale, bias, relu):
    g = torch.Generator(device="cuda").manual_seed(S * 7 + K)
    layer = _layer(g, S, K, n, m, 0.6)
    ld, ldr = (N + 7) // 8 * 8, (N + 7) // 8 * 8 + 8
    X = torch.randn((K, ld), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16)
    res = torch.randn((S, ldr), generator=g, device="cuda").to(torch.bfloat16)
    sc = torch.rand(S, generator=g, device="cuda") + 0.5 if scale else None
    bs = torch.randn(S, generator=g, device="cuda") if bias else None
    out = []
    for ydt, tdt in ((crisp.Y_F32, torch.float32), (crisp.Y_BF16, torch.bfloat16)):
        Y = torch.full((S, ld), 7.0, dtype=tdt, device="cuda")
        r = res.to(tdt)
        code = crisp.crisp_spmm_forced(layer.desc, layer.row_ptr, layer.col_idx, layer.vals, layer.idx_words, X, N, ld, Y, ld,
                                       ydt, crisp.epilogue(sc, bs, r, ldr, bool(relu)), shape)
        torch.cuda.synchronize()
        assert crisp.kernel_code_fields(code)["family"] == ("xres" if shape == 13 else "xlds")
        out.append(Y)
    assert torch.equal(out[0][:, :N].to(torch.bfloat16), out[1][:, :N])
    assert bool((out[1][:, N:] == 7.0).all())      # nothing past the last column
