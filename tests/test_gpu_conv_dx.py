"""The image gradient taken straight from the codes (product and fold in one) against the calls it stands for: the
quantisers, the product that writes the column gradient, and its fold.  Same bits, for every form of the kernel (the tile's
shape and the bytes of a row of codes that an item takes), at sizes that end inside a tile or an item; and the weight
gradient that shares its launch, under several plans of the two."""
import pytest
import torch

import paper_2406_15102_amd as hlq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# Nb, H, W, C, O, k, stride, pad, dilation
CASES = [
    (32, 32, 33, 128, 32, 3, 1, 1, 1),     # 128 x 128 tiles, ragged pixels, 32 bytes a step
    (32, 32, 32, 124, 48, 4, 1, 1, 1),     # 64 bytes a step, 16 of them past the end; channels past the end
    (32, 32, 32, 256, 144, 3, 1, 0, 1),    # 128 bytes a step, a ragged second one; no padding
    (48, 37, 40, 56, 16, 3, 1, 1, 1),      # 256 x 64, rows of codes half a step long
    (48, 37, 40, 44, 80, 4, 1, 1, 1),      # 256 x 64, two steps of 64 bytes, the second ragged
    (32, 28, 28, 72, 272, 3, 1, 2, 1),     # 128 x 64, padding past the image, three steps of 128 bytes
    (16, 16, 16, 40, 32, 3, 1, 1, 1),      # 64 x 64
    (16, 24, 20, 104, 64, 3, 1, 2, 2),     # dilated
    (32, 33, 31, 64, 64, 3, 2, 1, 1),      # classes of pixels of different sizes
    (32, 30, 30, 72, 48, 5, 3, 2, 2),      # stride and dilation without a common factor
    (32, 30, 30, 64, 96, 4, 2, 1, 2),      # ... and with one: half of the classes have no tap
    (16, 40, 36, 64, 128, 3, 1, 1, 1),
]


def _geom(c):
    Nb, H, W, C, O, k, s, p, d = c
    return hlq.hlq_conv_geom(Nb=Nb, H=H, W=W, C=C, O=O, kh=k, kw=k, stride_h=s, stride_w=s, pad_h=p, pad_w=p, dil_h=d, dil_w=d)


@pytest.mark.parametrize("c", CASES)
@pytest.mark.parametrize("dtype,flags", [(torch.bfloat16, 0), (torch.float32, 0), (torch.bfloat16, hlq.HLQ_FLAG_GX_8BIT),
                                         (torch.float32, hlq.HLQ_FLAG_GX_UNPACKED | hlq.HLQ_FLAG_SEPARATE_PRODUCTS)])
def test_image_gradient_is_the_fold_of_the_column_gradient(c, dtype, flags):
    Nb, H, W, C, O, k, s, p, d = c
    B, r, seed = 16, 8, 3
    geom = _geom(c)
    Ho, Wo, N, I = hlq.hlq_conv_sizes(geom)
    while N % B or N // B * r % 8 or I % 8:
        Nb *= 2
        assert Nb <= 1024
        geom = _geom((Nb,) + c[1:])
        Ho, Wo, N, I = hlq.hlq_conv_sizes(geom)
    print("conv", c, dtype, flags, "N", N, "I", I, flush=True)
    gen = torch.Generator(device=DEV).manual_seed(11)
    X, Wt, G = (torch.randn(shape, generator=gen, device=DEV).mul_(scale).to(dtype)
                for shape, scale in (((Nb, H, W, C), 1.0), ((O, k, k, C), 0.02), ((Nb, Ho, Wo, O), 1e-3)))
    bits = hlq.HLQ_BITS_8 if flags & hlq.HLQ_FLAG_GX_8BIT else hlq.HLQ_BITS_4
    Gq, Wq = torch.empty((N, O), dtype=torch.int8, device=DEV), torch.empty((I, O), dtype=torch.int8, device=DEV)
    sG, sW = torch.empty(N, dtype=torch.float32, device=DEV), torch.empty(I, dtype=torch.float32, device=DEV)
    ws = torch.empty(hlq.hlq_quantize_w_workspace_bytes(O, I), dtype=torch.uint8, device=DEV)
    hlq.hlq_quantize_g(G.reshape(N, O), B, seed, Gq, sG, None, bits)
    hlq.hlq_quantize_w(Wt.reshape(O, I), B, seed, Wq, sW, ws, None, bits)
    cols = torch.empty((N, I), dtype=dtype, device=DEV)
    hlq.hlq_int8_gemm_nt(Gq, Wq, sG, sW, 1.0 / B, cols)
    want = torch.full_like(X, 7.0)
    hlq.hlq_col2im(cols, geom, want)
    memory = torch.full((hlq.hlq_conv_workspace_bytes(geom, B, r, hlq.binding._dt(G), flags),), 0xFF, dtype=torch.uint8, device=DEV)
    dX, dW, only = torch.full_like(X, 3.0), torch.empty_like(Wt), torch.full_like(X, 5.0)
    hlq.hlq_conv2d_backward(G, X, Wt, geom, B, r, seed, flags, dX, dW, memory)
    hlq.hlq_conv2d_backward(G, None, Wt, geom, B, r, seed, flags, only, None, memory)
    assert torch.equal(dX, want) and torch.equal(only, want)
    # the column gradient's place in the scratch (the first thing in it where the image is projected straight) is untouched
    if C % 8 == 0:
        assert bool((memory[:cols.numel() * cols.element_size()] == 0xFF).all())
    assert torch.isfinite(dW.float()).all()


@pytest.mark.parametrize("c", [CASES[i] for i in (0, 2, 3, 5, 6, 7, 8, 11)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_weights_that_are_not_finite_stay_in_the_pixels_that_meet_them(c, dtype):
    """An infinite weight makes its column's scale infinite.  A pixel that does not have that column's tap gets nothing
    from it, not 0 * inf; one that has it gets what the fold of the column gradient gives, whatever the codes are."""
    Nb, H, W, C, O, k, s, p, d = c
    B, r, seed = 16, 8, 3
    geom = _geom(c)
    Ho, Wo, N, I = hlq.hlq_conv_sizes(geom)
    while N % B:
        Nb *= 2
        geom = _geom((Nb,) + c[1:])
        Ho, Wo, N, I = hlq.hlq_conv_sizes(geom)
    print("conv", c, dtype, "N", N, "I", I, flush=True)
    gen = torch.Generator(device=DEV).manual_seed(12)
    Wt, G = (torch.randn(shape, generator=gen, device=DEV).mul_(scale).to(dtype) for shape, scale in (((O, k, k, C), 0.02), ((Nb, Ho, Wo, O), 1e-3)))
    Wt[1, 0, 0, 5] = float("inf")
    Wt[2, k - 1, k - 1, C - 1] = -float("inf")
    Wt[0, k // 2, 0, C // 2] = float("nan")
    G[0, 0] = 0.0                                  # rows of codes whose scale is 0: 0 * inf where they are met
    G[1, Ho - 1, Wo - 1, 3] = float("inf")
    Gq, Wq = torch.empty((N, O), dtype=torch.int8, device=DEV), torch.empty((I, O), dtype=torch.int8, device=DEV)
    sG, sW = torch.empty(N, dtype=torch.float32, device=DEV), torch.empty(I, dtype=torch.float32, device=DEV)
    ws = torch.empty(hlq.hlq_quantize_w_workspace_bytes(O, I), dtype=torch.uint8, device=DEV)
    hlq.hlq_quantize_g(G.reshape(N, O), B, seed, Gq, sG, None, hlq.HLQ_BITS_4)
    hlq.hlq_quantize_w(Wt.reshape(O, I), B, seed, Wq, sW, ws, None, hlq.HLQ_BITS_4)
    assert not torch.isfinite(sW).all() and float(sG[0]) == 0.0
    cols = torch.empty((N, I), dtype=dtype, device=DEV)
    hlq.hlq_int8_gemm_nt(Gq, Wq, sG, sW, 1.0 / B, cols)
    want, dX = (torch.full((Nb, H, W, C), v, dtype=dtype, device=DEV) for v in (7.0, 3.0))
    hlq.hlq_col2im(cols, geom, want)
    hlq.hlq_conv2d_backward(G, None, Wt, geom, B, r, seed, 0, dX, None)
    assert not torch.isfinite(want).all() and torch.isfinite(want).any()
    assert torch.equal(dX.isnan(), want.isnan()) and torch.equal(dX.nan_to_num(nan=0.5), want.nan_to_num(nan=0.5))


def _time(run):
    for _ in range(3):
        run()
    times = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(4):
            run()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return sorted(times)[2]


def test_long_reduction_beside_a_full_chip_is_split():
    """490 tiles of the image gradient beside 15 of the weight gradient whose reduction takes 980 steps: left whole, for
    want of room beside the 490, they take 2.3 times as long as in 16 parts.  The plan's choice is held to 1.5 times."""
    geom = hlq.hlq_conv_geom(Nb=40, H=56, W=56, C=24, O=384, kh=5, kw=5, stride_h=1, stride_w=1, pad_h=2, pad_w=2, dil_h=1, dil_w=1)
    gen = torch.Generator(device=DEV).manual_seed(1)
    X, Wt, G = (torch.randn(shape, generator=gen, device=DEV) for shape in ((40, 56, 56, 24), (384, 5, 5, 24), (40, 56, 56, 384)))
    dX, dW = torch.empty_like(X), torch.empty_like(Wt)
    took = []
    try:
        for splits in (0, 16):
            hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, splits)
            ws = torch.empty(hlq.hlq_conv_workspace_bytes(geom, 16, 8, hlq.HLQ_F32, 0), dtype=torch.uint8, device=DEV)
            took.append(_time(lambda: hlq.hlq_conv2d_backward(G, X, Wt, geom, 16, 8, 3, 0, dX, dW, ws)))
    finally:
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, 0)
    print("us a pass: the plan's choice %.0f, 16 splits %.0f" % (took[0] * 250, took[1] * 250), flush=True)
    assert took[0] < 1.5 * took[1]


@pytest.mark.parametrize("c,stored", [((64, 14, 14, 384, 96, 8, 1, 0, 1), True), ((64, 14, 14, 384, 96, 5, 1, 0, 1), False)])
def test_tiles_that_fill_a_compute_unit_are_counted_one_to_a_unit(c, stored):
    """294 tiles of 64 taps over 96 codes, 97 KB of LDS each: two rounds of the chip, not one, and 1.7 times as long as the
    column gradient, which is stored then (the first thing in the scratch).  With 25 taps two fit a compute unit."""
    geom = _geom(c)
    _, _, N, I = hlq.hlq_conv_sizes(geom)
    Nb, H, W, C, O, k, *_ = c
    gen = torch.Generator(device=DEV).manual_seed(2)
    X, Wt, G = (torch.randn(shape, generator=gen, device=DEV).to(torch.bfloat16) for shape in ((Nb, H, W, C), (O, k, k, C), (N, O)))
    memory = torch.full((hlq.hlq_conv_workspace_bytes(geom, 16, 8, hlq.HLQ_BF16, 0),), 0xFF, dtype=torch.uint8, device=DEV)
    dX, dW = torch.empty_like(X), torch.empty_like(Wt)
    hlq.hlq_conv2d_backward(G, X, Wt, geom, 16, 8, 3, 0, dX, dW, memory)
    untouched = bool((memory[:N * I * 2] == 0xFF).all())
    assert untouched != stored


# Nb, H, W, C, O, k, stride, pad, dilation, B: the forms of the kernel that the cases above leave out, blocks of 32 and 64
# rows, and plans of the launch on either side of the 512 workgroups that are resident at once
PAIRS = [
    (16, 16, 16, 128, 256, 3, 2, 1, 1, 16),    # 64 x 64, two items of 128 bytes a tap; dW not split
    (16, 16, 16, 128, 144, 3, 2, 1, 1, 16),    # ... the second one ragged
    (16, 40, 36, 64, 32, 3, 1, 1, 1, 16),      # 128 x 64, items of 32 bytes; dW in 16 parts
    (16, 32, 32, 40, 32, 3, 1, 1, 1, 32),      # 64 x 64, items of 32 bytes, channels past the end
    (24, 20, 20, 40, 64, 5, 2, 2, 1, 32),      # 64 x 64, items of 64 bytes, stride
    (72, 16, 16, 128, 320, 3, 1, 1, 1, 64),    # 128 x 64, three items of 128 bytes, the last one half
    (64, 14, 14, 256, 256, 3, 1, 1, 1, 16),    # 500 workgroups in three parts
    (32, 32, 32, 256, 144, 3, 1, 0, 1, 16),    # more than 512, dW's first (bf16 projections)
    (156, 20, 20, 32, 32, 5, 1, 2, 1, 32),     # dW's reduction longer than the image gradient: more than there is room for
    (32, 32, 32, 124, 48, 4, 1, 1, 1, 16),     # the column matrix is stored
    (48, 37, 40, 44, 80, 4, 1, 1, 1, 16),
]


@pytest.mark.parametrize("c", PAIRS)
@pytest.mark.parametrize("dtype,flags,splits", [(torch.bfloat16, 0, 0), (torch.float32, 0, 3), (torch.bfloat16, hlq.HLQ_FLAG_GW_INT8, 0),
                                                (torch.float32, hlq.HLQ_FLAG_GW_INT8, 3), (torch.bfloat16, hlq.HLQ_FLAG_GW_INT8, 2)])
def test_both_gradients_of_one_launch(c, dtype, flags, splits):
    """dX against the three calls, and dW: integer projections bit for bit against the call for dW alone, bf16 ones against
    their product in 64 bits.  splits: parts of dW's reduction, 0 = the plan's choice."""
    Nb, H, W, C, O, k, s, p, d, B = c
    r, seed = B // 2, 4
    geom = _geom((Nb,) + c[1:9])
    Ho, Wo, N, I = hlq.hlq_conv_sizes(geom)
    while N % B or N // B * r % 16:
        Nb *= 2
        geom = _geom((Nb,) + c[1:9])
        Ho, Wo, N, I = hlq.hlq_conv_sizes(geom)
    print("conv", c, dtype, flags, splits, "N", N, "I", I, flush=True)
    gen = torch.Generator(device=DEV).manual_seed(13)
    X, Wt, G = (torch.randn(shape, generator=gen, device=DEV).mul_(scale).to(dtype)
                for shape, scale in (((Nb, H, W, C), 1.0), ((O, k, k, C), 0.02), ((Nb, Ho, Wo, O), 1e-3)))
    Gq, Wq = torch.empty((N, O), dtype=torch.int8, device=DEV), torch.empty((I, O), dtype=torch.int8, device=DEV)
    sG, sW = torch.empty(N, dtype=torch.float32, device=DEV), torch.empty(I, dtype=torch.float32, device=DEV)
    ws = torch.empty(hlq.hlq_quantize_w_workspace_bytes(O, I), dtype=torch.uint8, device=DEV)
    hlq.hlq_quantize_g(G.reshape(N, O), B, seed, Gq, sG, None, hlq.HLQ_BITS_4)
    hlq.hlq_quantize_w(Wt.reshape(O, I), B, seed, Wq, sW, ws, None, hlq.HLQ_BITS_4)
    cols = torch.empty((N, I), dtype=dtype, device=DEV)
    hlq.hlq_int8_gemm_nt(Gq, Wq, sG, sW, 1.0 / B, cols)
    want = torch.full_like(X, 7.0)
    hlq.hlq_col2im(cols, geom, want)
    dX, dW = torch.full_like(X, 3.0), torch.full_like(Wt, float("nan"))
    try:
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, splits)
        memory = torch.full((hlq.hlq_conv_workspace_bytes(geom, B, r, hlq.binding._dt(G), flags),), 0xFF, dtype=torch.uint8, device=DEV)
        hlq.hlq_conv2d_backward(G, X, Wt, geom, B, r, seed, flags, dX, dW, memory)
        torch.cuda.synchronize()
    finally:
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, 0)
    assert torch.equal(dX, want)
    # the column gradient's place, behind that of a column matrix that is stored, is untouched
    size = cols.numel() * cols.element_size()
    at = (size + 255) // 256 * 256 if C % (128 // B) else 0
    untouched = bool((memory[at:at + size] == 0xFF).all())
    assert untouched
    if flags & hlq.HLQ_FLAG_GW_INT8:
        alone = torch.full_like(Wt, 5.0)
        hlq.hlq_conv2d_backward(G, X, None, geom, B, r, seed, flags, None, alone)
        assert torch.equal(dW, alone)
        return
    hlq.hlq_im2col(X, geom, cols)
    Gh, Xh = (torch.empty((n, N // B * r), dtype=torch.bfloat16, device=DEV) for n in (O, I))
    hlq.hlq_hla_project_basis(G.reshape(N, O), B, r, hlq.HLQ_BASIS_NATURAL, Gh)
    hlq.hlq_hla_project_basis(cols, B, r, hlq.HLQ_BASIS_NATURAL, Xh)
    ref, size = Gh.double() @ Xh.double().T / B, Gh.double().abs() @ Xh.double().abs().T / B
    # products of bf16 are exact in fp32, Kc of them are summed in fp32, scaled, and rounded to the type (half a unit in
    # the last place of bf16 is up to 2^-8 of the value)
    eps = 2.0 ** -24 if dtype == torch.float32 else 2.0 ** -8
    assert torch.all((dW.reshape(O, I).double() - ref).abs() <= ref.abs() * (eps + 2.0 ** -22) + size * (N // B * r) * 2.0 ** -24)
