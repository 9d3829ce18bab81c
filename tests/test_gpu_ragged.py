"""Products whose K is no multiple of 16 or whose column count is none of 4: the register kernels with ranged resources
(the automatic choice) against the generic kernel (forced shape 4).  X carries NaN past its last row and column, Y a
guard band, so that a read or write past the edges shows."""
import pytest
import torch

from paper_2311_14272_amd import crisp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(1, 4), (2, 4), (3, 4), (4, 4), (1, 8), (2, 8), (4, 8), (8, 8)])
@pytest.mark.parametrize("B", [32, 64])
@pytest.mark.parametrize("S,K,N", [(5, 9, 1), (64, 16, 3), (203, 459, 66), (70, 147, 131), (130, 1000, 1), (33, 1001, 257),
                                   (96, 640, 2049), (2100, 72, 510)])
@pytest.mark.parametrize("ep,topk", [(0, 0), (1, 0), (1, 1)])
def test_ragged_product(n, m, B, S, K, N, ep, topk):
    g = torch.Generator(device="cuda").manual_seed(S + K + N)
    mode = crisp.LAYER_TOPK if topk else crisp.ROW_UNIFORM
    layer = crisp.alloc_layer(crisp.layer_desc(S, K, n, m, B, 0.6, crisp.SAL_MAG, mode))
    W = (torch.randn((S, K), generator=g, device="cuda") * 0.1).to(torch.bfloat16).view(torch.int16)
    crisp.prune_and_pack(layer, W, None)
    ld = (N + 7) // 8 * 8
    Xf = torch.full((K + 80, ld), float("nan"), dtype=torch.bfloat16, device="cuda")
    Xf[:K, :N] = torch.randn((K, N), generator=g, device="cuda").to(torch.bfloat16)
    X = Xf.view(torch.int16)
    sc = torch.rand(S, generator=g, device="cuda") + 0.5
    bs = torch.randn(S, generator=g, device="cuda")
    res = torch.full((S, ld + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    res[:, :N] = torch.randn((S, N), generator=g, device="cuda").to(torch.bfloat16)

    def product(dtype, shape):
        Y = torch.full((S + 1, ld), 7.0, dtype=dtype, device="cuda")
        r = res.to(dtype)
        e = crisp.epilogue(sc, bs, r, ld + 8, True) if ep else None
        code = crisp.crisp_spmm_forced(layer.desc, layer.row_ptr, layer.col_idx, layer.vals, layer.idx_words, X, N, ld, Y, ld,
                                       crisp.Y_BF16 if dtype == torch.bfloat16 else crisp.Y_F32, e, shape)
        torch.cuda.synchronize()
        assert bool((Y[S] == 7.0).all()) and bool((Y[:S, N:] == 7.0).all()), "guard band written"
        return Y[:S, :N], crisp.kernel_code_fields(code)["family"]

    ref, family = product(torch.float32, 4)
    assert family == "generic"
    y, family = product(torch.float32, crisp.SHAPE_AUTO)
    if K % 16 or N % 4:
        assert family == "reg"
    # the products are exact in fp32 and only their order differs: at most K roundings of 2^-24 of the sum of the
    # magnitudes, which the values here keep under 0.1 * K, plus those of the tail (outputs of about ten at most)
    assert float((y - ref).abs().max()) <= 2.0 ** -24 * (K * 0.1 * K * 0.6 + 64)
    yb, _ = product(torch.bfloat16, crisp.SHAPE_AUTO)
    assert torch.equal(y.to(torch.bfloat16), yb)


@pytest.mark.parametrize("n,m", [(1, 4), (2, 4), (3, 4), (2, 8), (4, 8)])
@pytest.mark.parametrize("B", [32, 64])
@pytest.mark.parametrize("S,K,N", [(70, 147, 131), (130, 1000, 257), (96, 640, 66)])
def test_forced_shapes(n, m, B, S, K, N):
    """Narrow strips and the split by four can be forced on ragged problems, with and without the sparse instruction;
    a shape that does not apply leaves the choice to the library, whose kernel and bits it then has."""
    g = torch.Generator(device="cuda").manual_seed(S + K + N)
    layer = crisp.alloc_layer(crisp.layer_desc(S, K, n, m, B, 0.6, crisp.SAL_MAG))
    W = (torch.randn((S, K), generator=g, device="cuda") * 0.1).to(torch.bfloat16).view(torch.int16)
    crisp.prune_and_pack(layer, W, None)
    ld = (N + 7) // 8 * 8
    X = torch.randn((K, ld), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16)

    def product(shape):
        Y = torch.full((S, ld), float("nan"), dtype=torch.float32, device="cuda")
        code = crisp.crisp_spmm_forced(layer.desc, layer.row_ptr, layer.col_idx, layer.vals, layer.idx_words, X, N, ld, Y, ld,
                                       crisp.Y_F32, None, shape)
        torch.cuda.synchronize()
        f = crisp.kernel_code_fields(code)
        return Y[:, :N], (f["family"], f["shape"], f["sparse_mfma"])

    ref, kernel = product(4)
    assert kernel[0] == "generic"
    auto, chosen = product(crisp.SHAPE_AUTO)
    sparse = int(n <= 2)
    for shape, want in ((1, ("reg", 1, 0)), (2, ("reg", 2, 0)), (8, ("reg", 1, sparse)), (9, ("reg", 2, sparse))):
        y, kernel = product(shape)
        assert kernel == want, shape
        # (the bound of test_ragged_product)
        assert float((y - ref).abs().max()) <= 2.0 ** -24 * (K * 0.1 * K * 0.6 + 64), shape
    for shape in (0, 3, 5, 6, 7, 10, 13, 15, 16, 17, 18):
        y, kernel = product(shape)
        assert kernel == chosen, shape
        assert torch.equal(y, auto), shape


@pytest.mark.parametrize("n,m", [(1, 4), (2, 4), (3, 4), (4, 4), (1, 8), (2, 8), (4, 8), (8, 8)])
@pytest.mark.parametrize("B", [32, 64])
@pytest.mark.parametrize("K,N", [(129, 66), (163, 7), (1000, 130)])
def test_infinite_activations(n, m, B, K, N):
    """An infinite element of X: wherever the generic kernel's result is a number or an infinity, the ragged register
    kernels have the same infinity or a number within the bound of test_ragged_product.  The last row of X, which lies
    in a short group for two of the sizes, is among the infinite ones."""
    S = 96
    g = torch.Generator(device="cuda").manual_seed(K + N)
    layer = crisp.alloc_layer(crisp.layer_desc(S, K, n, m, B, 1.0, crisp.SAL_MAG))
    W = (torch.randn((S, K), generator=g, device="cuda") * 0.1).to(torch.bfloat16).view(torch.int16)
    crisp.prune_and_pack(layer, W, None)
    ld = (N + 7) // 8 * 8
    Xf = torch.randn((K, ld), generator=g, device="cuda")
    for i, k in enumerate(list(range(0, K, 17)) + [K - 1]):
        Xf[k, i % N] = float("inf") if i % 2 else float("-inf")       # few rows per column: most have one at most
    X = Xf.to(torch.bfloat16).view(torch.int16)

    def product(shape):
        Y = torch.zeros((S, ld), dtype=torch.float32, device="cuda")
        code = crisp.crisp_spmm_forced(layer.desc, layer.row_ptr, layer.col_idx, layer.vals, layer.idx_words, X, N, ld, Y, ld,
                                       crisp.Y_F32, None, shape)
        torch.cuda.synchronize()
        return Y[:, :N], crisp.kernel_code_fields(code)["family"]

    ref, family = product(4)
    assert family == "generic"
    assert bool(torch.isinf(ref).any())
    inf, fin = torch.isinf(ref), torch.isfinite(ref)
    for shape in (crisp.SHAPE_AUTO, 1, 2, 8, 9):
        y, family = product(shape)
        assert family == "reg"
        assert torch.equal(y[inf], ref[inf]), "shape %d: %d of %d infinities lost" % (shape, int((y[inf] != ref[inf]).sum()), int(inf.sum()))
        if bool(fin.any()):
            assert float((y[fin] - ref[fin]).abs().max()) <= 2.0 ** -24 * (K * 0.1 * K * 0.6 + 64), shape


# S, K, N, n, m, density, bf16: on many tiles with 32x32 blocks and the sparse instruction the generic kernel stays for long
# rows, fp32 output and 1:8 (us of the register kernels / generic: 72 / 47, 205 / 139, 221 / 185), else it does not
@pytest.mark.parametrize("case,family", [((699, 4401, 5100, 1, 8, 0.2, 1), "generic"), ((1112, 2616, 3553, 2, 4, 1.0, 0), "generic"),
                                         ((1102, 541, 20837, 1, 8, 0.3, 0), "generic"), ((203, 459, 25003, 2, 4, 0.5, 1), "reg"),
                                         ((64, 147, 70001, 1, 8, 0.5, 0), "reg")], ids=str)
def test_choice_with_32_row_blocks(case, family):
    S, K, N, n, m, dens, bf16 = case
    g = torch.Generator(device="cuda").manual_seed(S)
    layer = crisp.alloc_layer(crisp.layer_desc(S, K, n, m, 32, dens, crisp.SAL_MAG))
    W = (torch.randn((S, K), generator=g, device="cuda") * 0.05).to(torch.bfloat16).view(torch.int16)
    crisp.prune_and_pack(layer, W, None)
    ld = (N + 7) // 8 * 8
    X = torch.randn((K, ld), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16)
    out = []
    for shape in (crisp.SHAPE_AUTO, 4):
        Y = torch.full((S, ld), float("nan"), dtype=torch.bfloat16 if bf16 else torch.float32, device="cuda")
        code = crisp.crisp_spmm_forced(layer.desc, layer.row_ptr, layer.col_idx, layer.vals, layer.idx_words, X, N, ld, Y, ld,
                                       crisp.Y_BF16 if bf16 else crisp.Y_F32, None, shape)
        torch.cuda.synchronize()
        out.append((crisp.kernel_code_fields(code)["family"], Y[:, :N].float()))
    assert out[0][0] == family and out[1][0] == "generic"
    # the same products in another order, and for bf16 the roundings of either (1.66e-3 each of a result)
    assert float((out[0][1] - out[1][1]).norm() / out[1][1].norm()) <= (2 * 1.66e-3 if bf16 else 1e-5)


# 1:8, 32x32 blocks, long rows: the generic kernel's wide strips are ahead with a layer tail as well (us of the register
# kernels / generic: 130 / 104, 221 / 184, 50 / 42), but not on fewer tiles, more tiles or shorter rows
@pytest.mark.parametrize("case,ep,family", [((64, 4080, 65793, 0.4, 1), 1, "generic"), ((64, 3848, 69759, 0.75, 0), 1, "generic"),
                                            ((64, 1224, 68186, 0.53, 1), 1, "generic"), ((64, 4080, 40001, 0.4, 1), 1, "reg"),
                                            ((64, 1224, 68186, 0.25, 1), 1, "reg"), ((128, 1224, 68186, 0.53, 1), 1, "reg")], ids=str)
def test_choice_for_one_of_eight(case, ep, family):
    S, K, N, dens, bf16 = case
    g = torch.Generator(device="cuda").manual_seed(S)
    layer = crisp.alloc_layer(crisp.layer_desc(S, K, 1, 8, 32, dens, crisp.SAL_MAG))
    W = (torch.randn((S, K), generator=g, device="cuda") * 0.05).to(torch.bfloat16).view(torch.int16)
    crisp.prune_and_pack(layer, W, None)
    ld = (N + 7) // 8 * 8
    X = torch.randn((K, ld), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16)
    sc, bs = torch.rand(S, generator=g, device="cuda") + 0.5, torch.randn(S, generator=g, device="cuda")
    out = []
    for shape in (crisp.SHAPE_AUTO, 4):
        Y = torch.full((S, ld), float("nan"), dtype=torch.bfloat16 if bf16 else torch.float32, device="cuda")
        code = crisp.crisp_spmm_forced(layer.desc, layer.row_ptr, layer.col_idx, layer.vals, layer.idx_words, X, N, ld, Y, ld,
                                       crisp.Y_BF16 if bf16 else crisp.Y_F32, crisp.epilogue(sc, bs, None, 0, True) if ep else None, shape)
        torch.cuda.synchronize()
        out.append((crisp.kernel_code_fields(code)["family"], Y[:, :N].float()))
    assert out[0][0] == family and out[1][0] == "generic"
    # the same products in another order, and for bf16 the roundings of either (1.66e-3 each of a result)
    assert float((out[0][1] - out[1][1]).norm() / out[1][1].norm()) <= (2 * 1.66e-3 if bf16 else 1e-5)
