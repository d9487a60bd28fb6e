"""Products whose last columns fill no tile: the values that an epilogue keeps over its guarded stores.
The compiler may put one back, from the other half of the register file, at the end of the guarded region, where the lanes
past the last column were still switched off: their later rows were scaled by what had been there.  Every kernel that a pair of
products can take is held to the integer product of the codes in 64 bits."""
import pytest
import torch

import paper_2406_15102_amd as hlq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GWI, X8 = hlq.HLQ_FLAG_GW_INT8, hlq.HLQ_FLAG_GX_8BIT
B, r, SEED = 16, 8, 3


def _codes(T, tensor):
    N, D = T.shape
    q, s = torch.empty((D, N // B * r), dtype=torch.int8, device=DEV), torch.empty(D, device=DEV)
    ws = torch.empty(hlq.hlq_hla_quantize_workspace_bytes(D), dtype=torch.uint8, device=DEV)
    hlq.hlq_hla_quantize(T, B, r, SEED, tensor, q, s, ws)
    return q, s


def _product(a, sa, b, sb):
    return (a.double() @ b.double().t()) * (sa.double()[:, None] * sb.double()[None, :] / B)


# 2040 = 7 x 256 + 248 (128-tiles: 15 x 128 + 120), 2020 ends inside 16 bytes of bf16, 1944 and 1800 leave the last wavefront's
# columns partly or wholly empty; rows that end inside a tile too
@pytest.mark.parametrize("N,I,O", [(2848, 2040, 2304), (1632, 1944, 2064), (2080, 1800, 1296), (544, 520, 272)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("store", [False, True])
def test_columns_at_the_edge(N, I, O, dtype, store):
    g = torch.Generator(device=DEV).manual_seed(N)
    G, X, W = (torch.randn(s, generator=g, device=DEV).to(dtype) for s in ((N, O), (N, I), (O, I)))
    (gq, sg), (xq, sx) = _codes(G, 3), _codes(X, 2)
    want_w = _product(gq, sg, xq, sx)
    rel = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -21       # one rounding of the output, three of the scales and the product
    for flags in (X8 | GWI, GWI):
        bits = hlq.HLQ_BITS_8 if flags & X8 else hlq.HLQ_BITS_4
        q, s = torch.empty((N, O), dtype=torch.int8, device=DEV), torch.empty(N, device=DEV)
        hlq.hlq_quantize_g(G, B, SEED, q, s, None, bits)
        wq, sw = torch.empty((I, O), dtype=torch.int8, device=DEV), torch.empty(I, device=DEV)
        hlq.hlq_quantize_w(W, B, SEED, wq, sw, torch.empty(hlq.hlq_quantize_w_workspace_bytes(O, I), dtype=torch.uint8, device=DEV), None, bits)
        want_x = _product(q, s, wq, sw)
        try:
            for tile in (0, 128, 256):
                for direct in (1, 0):
                    hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_TILE, tile)
                    hlq.hlq_set_option(hlq.HLQ_OPT_DIRECT_TO_LDS, direct)
                    dX, dW = torch.empty((N, I), dtype=dtype, device=DEV), torch.empty((O, I), dtype=dtype, device=DEV)
                    ws = torch.empty(hlq.hlq_workspace_bytes_mode(N, I, O, B, r, store, flags), dtype=torch.uint8, device=DEV)
                    hlq.hlq_linear_backward_mode(G, None if store else X, xq if store else None, sx if store else None, W, N, I, O, B, r, SEED,
                                                 flags, dX, dW, ws)
                    torch.cuda.synchronize()
                    for got, want in ((dX, want_x), (dW, want_w)):
                        assert ((got.double() - want).abs() <= rel * want.abs()).all(), (flags, tile, direct)
        finally:
            hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_TILE, 0)
            hlq.hlq_set_option(hlq.HLQ_OPT_DIRECT_TO_LDS, 1)
