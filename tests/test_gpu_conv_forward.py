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


def _infinities(act):
    """Few infinite elements, of both signs, none two in one filter window of the same image where images are large."""
    flat = act.view(act.shape[0], act.shape[1], -1)
    for c in range(0, flat.shape[0], 7):
        flat[c, c % flat.shape[1], (c * 37 + 5) % flat.shape[2]] = float("inf") if c % 2 else float("-inf")


@pytest.mark.parametrize("n,m", [(1, 4), (2, 4), (3, 4), (1, 8), (2, 8), (4, 8)])
@pytest.mark.parametrize("shape,family", [
    ((96, 128, 13, 13, 45, 3, 1, 1, 64, 1.0), "conv_lds"),     # odd number of columns
    ((64, 72, 33, 33, 13, 3, 1, 1, 64, 1.0), "conv_lds"),      # ... channels that are no multiple of the block edge
    ((40, 64, 7, 7, 301, 5, 1, 2, 32, 1.0), "conv_lds"),
    ((512, 40, 18, 18, 90, 3, 2, 1, 64, 1.0), "conv_lds"),     # K no multiple of 16
    ((320, 40, 13, 13, 2, 1, 2, 0, 64, 1.0), "reg"),           # strided, one tap: rows located one by one
    ((160, 27, 13, 13, 2, 1, 2, 0, 64, 1.0), "reg"),           # ... with a short last group
    ((192, 64, 13, 13, 2, 1, 2, 0, 64, 1.0), "reg"),           # columns one by one
    ((1100, 128, 10, 4, 3, 1, 2, 0, 64, 1.0), "reg"),          # pairs from one 8-byte piece
    ((300, 96, 13, 13, 2, 1, 2, 0, 32, 0.7), "reg"),
    ((192, 64, 13, 13, 2, 3, 2, 1, 64, 0.6), "reg"),           # several taps
], ids=str)
def test_infinite_activations(shape, family, n, m):
    """Convolutions whose K is no multiple of 16 or whose column count is none of four: wherever the product over X (generic
    kernel) is a number or an infinity, the fused kernel that runs in its place has the same infinity, or a number within the
    bound of the sums' order."""
    S, C, H, W, batch, k, stride, pad, B, dens = shape
    c = Conv(S, C, H, W, batch, k, stride, pad, n, m, B, dens, act=_infinities)
    assert c.plan == "im2col" and (c.cv.K % 16 or c.N % 4)
    out, way, ran = c.forward()
    ref = c.through_x()
    inf, fin = torch.isinf(ref), torch.isfinite(ref)
    print(shape, n, m, way, ran, int(inf.sum()), int((out[inf] != ref[inf]).sum()), flush=True)
    assert bool(inf.any()) and bool(fin.any())
    assert torch.equal(out[inf], ref[inf]), "%s: %d of %d infinities lost" % (ran, int((out[inf] != ref[inf]).sum()), int(inf.sum()))
    bound = 2.0 ** -24 * c.cv.K * (c.W.view(torch.bfloat16).float().abs().sum(1).max().item() * 5 + 1)
    assert float((out[fin] - ref[fin]).abs().max()) <= bound
    assert ran == family or (ran is None and (n, m) not in ((1, 4), (2, 8)))       # dense patterns may stay with X


@pytest.mark.parametrize("n,m", [(1, 4), (2, 4), (3, 4), (4, 4), (1, 8), (2, 8), (4, 8), (8, 8)])
@pytest.mark.parametrize("shape", [(300, 272, 28, 28, 2, 3, 2, 0, 64, 1.0), (70, 400, 16, 16, 2, 3, 1, 0, 32, 1.0)], ids=str)
def test_infinite_weights_over_several_chunks(shape, n, m):
    """Channels in several chunks, block columns of several taps: an infinite weight meets its own activations only, whatever
    chunk its block is walked in."""
    S, C, H, W, batch, k, stride, pad, B, dens = shape

    def weight(Wf):
        for i in range(0, Wf.shape[0], 3):
            Wf[i, (i * 131 + 17) % Wf.shape[1]] = float("inf") if i % 2 else float("-inf")

    c = Conv(S, C, H, W, batch, k, stride, pad, n, m, B, dens, weight=weight)
    y, ref = c.layer, c.through_x()
    Y = torch.full((S, c.ld), float("nan"), dtype=torch.float32, device="cuda")
    code = crisp.crisp_conv_spmm_forced(y.desc, crisp.conv_desc_of(c.cv), y.row_ptr, y.col_idx, y.vals, y.idx_words, c.act, Y, c.ld,
                                        crisp.Y_F32, None, 19)
    torch.cuda.synchronize()
    f = crisp.kernel_code_fields(code)
    assert f["family"] == "conv_lds" and f["shape"] in (1, 2)
    out = Y[:, :c.N]
    inf, fin = torch.isinf(ref), torch.isfinite(ref)
    print(shape, n, m, int(inf.sum()), int(torch.isnan(out[inf]).sum()), flush=True)
    assert bool(inf.any()) and bool(fin.any()) and not bool(torch.isnan(ref).any())
    assert torch.equal(out[inf], ref[inf]), "%d of %d infinities lost" % (int((out[inf] != ref[inf]).sum()), int(inf.sum()))
    rows = c.W.view(torch.bfloat16).float().abs()
    bound = 2.0 ** -24 * c.cv.K * (rows[torch.isfinite(rows).all(1)].sum(1).max().item() * 5 + 1)
    assert float((out[fin] - ref[fin]).abs().max()) <= bound


# us of the ways: through X, from a window, in the register kernels
@pytest.mark.parametrize("shape,uneven,expect", [
    ((256, 464, 28, 28, 3, 5, 1, 2, 1, 4, 32, 0.70), 0, "im2col"),    # 62 / 100 / 149
    ((75, 304, 20, 20, 3, 1, 2, 0, 4, 8, 64, 0.47), 0, "im2col"),     # 8.8 / - / 12.8
    ((195, 352, 28, 28, 20, 5, 2, 2, 1, 4, 64, 0.47), 1, "im2col"),   # 57 / 84 / 129, block-rows of any length
    ((794, 384, 33, 33, 4, 3, 2, 1, 3, 4, 64, 0.77), 1, "im2col"),    # 42 / 65 / 102
    ((508, 64, 20, 20, 18, 3, 2, 1, 2, 4, 64, 0.77), 0, "reg"),       # planned fused: - / 15 / 8.1
    ((256, 192, 20, 20, 18, 5, 1, 2, 2, 8, 64, 0.32), 0, "reg"),      # - / 26.5 / 16.5
    ((512, 512, 14, 14, 256, 3, 2, 1, 4, 8, 64, 0.40), 0, "conv_lds"),   # 130 / 55 / -
    ((256, 256, 14, 14, 256, 3, 1, 1, 2, 8, 64, 0.60), 0, "conv_lds"),   # - / 39 / 47
    ((64, 64, 33, 33, 119, 3, 1, 1, 4, 8, 64, 0.281), 1, "conv_lds"),    # 67 / 17 / -, block-rows of any length
], ids=str)
def test_the_faster_way_is_taken(shape, uneven, expect):
    """Convolutions that once took the slower way by a third and more, and some that are well ahead in the window kernel."""
    S, C, H, W, batch, k, stride, pad, n, m, B, dens = shape
    cv = synth.ConvShape(C, H, W, batch, k, k, stride, pad)
    layer = crisp.alloc_layer(crisp.layer_desc(S, cv.K, n, m, B, dens, crisp.SAL_MAG, crisp.LAYER_TOPK if uneven else crisp.ROW_UNIFORM))
    g = torch.Generator(device="cuda").manual_seed(1)
    crisp.prune_and_pack(layer, torch.randn((S, cv.K), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16), None)
    act = torch.randn((C, batch, H, W), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16)
    ld = (cv.Ncol + 7) // 8 * 8
    X = torch.empty(max(8, crisp.conv_plan(layer.desc, cv)[1] // 2), dtype=torch.int16, device="cuda")
    Y = torch.empty((S, ld), dtype=torch.bfloat16, device="cuda")
    way = crisp.conv_forward(layer, cv, act, Y, ld, crisp.Y_BF16, X)
    if way == "fused":
        code = crisp.crisp_conv_spmm_forced(layer.desc, crisp.conv_desc_of(cv), layer.row_ptr, layer.col_idx, layer.vals, layer.idx_words,
                                            act, Y, ld, crisp.Y_BF16, None, crisp.SHAPE_CONV_FORWARD)
        way = crisp.kernel_code_fields(code)["family"]
    torch.cuda.synchronize()
    assert way == expect
