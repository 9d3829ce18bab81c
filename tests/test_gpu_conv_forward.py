"""Whole convolutions that are planned through a materialised X and run by a fused kernel: which one, and what that kernel
does where the product over X was already right."""
import pytest
import torch

from paper_2311_14272_amd import crisp, synth

pytestmark = pytest.mark.gpu


class Conv:
    """A convolution of random activations, its packed layer, and its product over X by the generic kernel."""

    def __init__(self, S, C, H, W, batch, k, stride, pad, n, m, B, dens, weight=None, act=None, hints=0):
        g = torch.Generator(device="cuda").manual_seed(S + C + H * 7 + n * 3 + m)
        self.cv = synth.ConvShape(C, H, W, batch, k, k, stride, pad)
        self.S, self.N = S, self.cv.Ncol
        self.layer = crisp.alloc_layer(crisp.layer_desc(S, self.cv.K, n, m, B, dens, crisp.SAL_MAG, crisp.ROW_UNIFORM, hints))
        Wf = torch.randn((S, self.cv.K), generator=g, device="cuda") * 0.1
        if weight is not None:
            weight(Wf)
        self.W = Wf.to(torch.bfloat16).view(torch.int16)
        crisp.prune_and_pack(self.layer, self.W, None)
        actf = torch.randn((C, batch, H, W), generator=g, device="cuda").abs() + 0.1
        if act is not None:
            act(actf)
        self.act = actf.to(torch.bfloat16).view(torch.int16)
        self.ld = (self.N + 7) // 8 * 8
        self.plan, nbytes = crisp.conv_plan(self.layer.desc, self.cv)
        self.X = torch.empty(nbytes // 2, dtype=torch.int16, device="cuda")

    def through_x(self):
        y = self.layer
        X = torch.empty((self.cv.K, self.ld), dtype=torch.int16, device="cuda")
        crisp.crisp_im2col(crisp.conv_desc_of(self.cv), self.act, X, self.ld)
        Y = torch.empty((self.S, self.ld), dtype=torch.float32, device="cuda")
        crisp.crisp_spmm_forced(y.desc, y.row_ptr, y.col_idx, y.vals, y.idx_words, X, self.N, self.ld, Y, self.ld, crisp.Y_F32, None, 4)
        torch.cuda.synchronize()
        return Y[:, :self.N]

    def forward(self):
        """The result, the way taken and (fused) the kernel family."""
        y = self.layer
        Y = torch.full((self.S, self.ld), float("nan"), dtype=torch.float32, device="cuda")
        way = crisp.conv_forward(y, self.cv, self.act, Y, self.ld, crisp.Y_F32, self.X)
        out, family = Y[:, :self.N].clone(), None
        if way == "fused":
            code = crisp.crisp_conv_spmm_forced(y.desc, crisp.conv_desc_of(self.cv), y.row_ptr, y.col_idx, y.vals, y.idx_words, self.act,
                                                Y, self.ld, crisp.Y_F32, None, crisp.SHAPE_CONV_FORWARD)
            family = crisp.kernel_code_fields(code)["family"]
            torch.cuda.synchronize()
            assert torch.equal(out.isnan(), Y[:, :self.N].isnan()) and torch.equal(out.nan_to_num(), Y[:, :self.N].nan_to_num())
        torch.cuda.synchronize()
        return out, way, family


@pytest.mark.parametrize("shape", [(746, 25, 14, 14, 2, 3, 1, 1, 2, 8, 64, 0.22), (320, 12, 14, 14, 1, 3, 1, 1, 2, 4, 64, 0.6),
                                   (256, 40, 14, 14, 1, 3, 1, 1, 4, 8, 64, 0.5)], ids=str)
def test_few_channels_in_the_register_kernels(shape):
    """The rule by which a planned X gives way weighs the register kernels; they are what then runs, and not the kernel for
    few channels, which takes a workgroup per 1024 output positions and image (746 x 225 x 392: 35.8 us against 10.6)."""
    c = Conv(*shape)
    out, way, family = c.forward()
    assert c.plan == "im2col" and way in ("fused", "im2col")
    assert family in (None, "reg", "conv_lds")
    ref = c.through_x()
    # exact products in fp32, in another order: at most K roundings of 2^-24 of the sum of the magnitudes (0.1 each)
    assert float((out - ref).abs().max()) <= 2.0 ** -24 * c.cv.K * (c.W.view(torch.bfloat16).float().abs().sum(1).max().item() * 5 + 1)
