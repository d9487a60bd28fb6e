"""Products whose last columns fill no tile: the values that an epilogue keeps over its guarded stores.
The compiler may put one back, from the other half of the register file, at the end of a guarded region inside another, where the
lanes past the last column were still switched off: their later rows were scaled by what had been there.  Every pair of kinds of
the two products, either product alone, k splits, and rows of bf16 that are only 8-byte aligned are held to the product in 64 bits."""
import pytest
import torch

import paper_2406_15102_amd as hlq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GWI, X8, SEP = hlq.HLQ_FLAG_GW_INT8, hlq.HLQ_FLAG_GX_8BIT, hlq.HLQ_FLAG_SEPARATE_PRODUCTS
B, r, SEED = 16, 8, 3


def _codes(T, tensor):
    N, D = T.shape
    q, s = torch.empty((D, N // B * r), dtype=torch.int8, device=DEV), torch.empty(D, device=DEV)
    ws = torch.empty(hlq.hlq_hla_quantize_workspace_bytes(D), dtype=torch.uint8, device=DEV)
    hlq.hlq_hla_quantize(T, B, r, SEED, tensor, q, s, ws)
    return q, s


def _projection(T):
    N, D = T.shape
    out = torch.empty((D, N // B * r), dtype=torch.bfloat16, device=DEV)
    hlq.hlq_hla_project(T, B, r, out)
    return out


def _product(a, sa, b, sb):
    return (a.double() @ b.double().t()) * (sa.double()[:, None] * sb.double()[None, :] / B)


# 2040 = 7 x 256 + 248 (128-tiles: 15 x 128 + 120), 1944 and 1800 leave the last wavefront's columns partly or wholly empty; rows
# that end inside a tile too.  The 4-bit codes of 288 out-features are kept as nibbles, those of 272 as bytes, of the others in the 6-bit layout.
@pytest.mark.parametrize("N,I,O", [(2848, 2040, 2304), (1632, 1944, 2064), (2080, 1800, 1296), (544, 520, 272), (1056, 1304, 288)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("store", [False, True])
@pytest.mark.parametrize("gw", [GWI, 0])
def test_columns_at_the_edge(N, I, O, dtype, store, gw):
    g = torch.Generator(device=DEV).manual_seed(N)
    G, X, W = (torch.randn(s, generator=g, device=DEV).to(dtype) for s in ((N, O), (N, I), (O, I)))
    rel = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -21       # one rounding of the output, three of the scales and the product
    if gw:
        (gq, sg), (xq, sx) = _codes(G, 3), _codes(X, 2)
        want_w, slack = _product(gq, sg, xq, sx), 0.0
    else:
        gq, xq, sx = _projection(G), _projection(X), None
        want_w = gq.double() @ xq.double().t() / B
        # sums of K products in fp32, in any order and split, cut off or rounded: a unit in the last place of the sum of magnitudes each
        slack = gq.shape[1] * 2.0 ** -23 * (gq.double().abs() @ xq.double().abs().t()) / B
    for gx in (X8, 0):
        bits = hlq.HLQ_BITS_8 if gx else hlq.HLQ_BITS_4
        q, s = torch.empty((N, O), dtype=torch.int8, device=DEV), torch.empty(N, device=DEV)
        hlq.hlq_quantize_g(G, B, SEED, q, s, None, bits)
        wq, sw = torch.empty((I, O), dtype=torch.int8, device=DEV), torch.empty(I, device=DEV)
        hlq.hlq_quantize_w(W, B, SEED, wq, sw, torch.empty(hlq.hlq_quantize_w_workspace_bytes(O, I), dtype=torch.uint8, device=DEV), None, bits)
        want_x = _product(q, s, wq, sw)
        try:
            for tile, direct, splits, sep in [(t, d, 0, 0) for t in (0, 128, 256) for d in (1, 0)] + [(128, 1, 3, 0), (256, 1, 2, 0), (0, 1, 0, SEP), (256, 1, 1, SEP), (128, 0, 2, SEP)]:
                hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_TILE, tile)
                hlq.hlq_set_option(hlq.HLQ_OPT_DIRECT_TO_LDS, direct)
                hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, splits)
                flags = gx | gw | sep
                dX, dW = torch.empty((N, I), dtype=dtype, device=DEV), torch.empty((O, I), dtype=dtype, device=DEV)
                ws = torch.empty(hlq.hlq_workspace_bytes_mode(N, I, O, B, r, store, flags), dtype=torch.uint8, device=DEV)
                hlq.hlq_linear_backward_mode(G, None if store else X, xq if store else None, sx if store else None, W, N, I, O, B, r, SEED,
                                             flags, dX, dW, ws)
                torch.cuda.synchronize()
                case = (flags, tile, direct, splits)
                assert ((dX.double() - want_x).abs() <= rel * want_x.abs()).all(), case
                assert ((dW.double() - want_w).abs() <= rel * want_w.abs() + (1 + rel) * slack).all(), case
        finally:
            for o, v in ((hlq.HLQ_OPT_PLAN_TILE, 0), (hlq.HLQ_OPT_DIRECT_TO_LDS, 1), (hlq.HLQ_OPT_PLAN_SPLITS, 0)):
                hlq.hlq_set_option(o, v)


# 2020 columns end inside 16 bytes of bf16: stores of 8 bytes, the last half missing.  Only the calls for one product take them.
@pytest.mark.parametrize("M,N,K", [(1000, 2020, 640), (300, 1804, 1056), (264, 132, 128)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_rows_of_half_pieces(M, N, K, dtype):
    g = torch.Generator(device=DEV).manual_seed(M)
    a, b = (torch.randint(-7, 8, s, generator=g, device=DEV, dtype=torch.int8) for s in ((M, K), (N, K)))
    sa, sb = (torch.rand(n, generator=g, device=DEV) + 0.5 for n in (M, N))
    want = (a.double() @ b.double().t()) * (sa.double()[:, None] * sb.double()[None, :] / B)
    packed = [(t[:, 0::2] & 15 | t[:, 1::2] << 4).view(torch.uint8).contiguous() for t in (a, b)]
    fa, fb = a.to(torch.bfloat16), b.to(torch.bfloat16)
    rel = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -21
    try:
        for tile in (0, 128, 256):
            for splits in (0, 2):
                hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_TILE, tile)
                hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, splits)
                for kind, call in enumerate((hlq.hlq_int8_gemm_nt, hlq.hlq_bf16_gemm_nt, hlq.hlq_int4_gemm_nt)):
                    # the words behind C stay what they are
                    room = torch.full((M * N + 64,), 7.0, dtype=dtype, device=DEV)
                    C = room[:M * N].view(M, N)
                    ws = torch.empty(max(16, hlq.hlq_gemm_workspace_bytes(kind, M, N, K)), dtype=torch.uint8, device=DEV)
                    if kind == 1:
                        call(fa, fb, 1.0 / B, C, ws)
                        ref = a.double() @ b.double().t() / B
                    else:
                        x, y = (a, b) if kind == 0 else packed
                        call(x, y, sa, sb, 1.0 / B, C, None, ws)
                        ref = want
                    torch.cuda.synchronize()
                    assert ((C.double() - ref).abs() <= rel * ref.abs()).all(), (kind, tile, splits)
                    assert (room[M * N:] == 7.0).all()
    finally:
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_TILE, 0)
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, 0)
