"""Projections that the whole path makes itself have rows padded to whole 128-byte steps of the dW product; a store that is
handed over has none.  Sums meet only zeros more, in the same order, so dW is the same bit for bit, whatever the scratch held
before; and scratch of the size without padding is still enough."""
import pytest
import torch

import paper_2406_15102_amd as hlq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GWI, X4 = hlq.HLQ_FLAG_GW_INT8, hlq.HLQ_FLAG_XC_INT4


def _inputs(N, I, O, dtype):
    g = torch.Generator(device=DEV).manual_seed(N + I + O)
    return [torch.randn(s, generator=g, device=DEV).to(dtype) for s in ((N, O), (N, I), (O, I))]


def _backward(G, X, Xc, sXc, W, I, B, r, flags, extra=0):
    N, O = G.shape
    dX, dW = torch.empty((N, I), dtype=G.dtype, device=DEV), torch.empty((O, I), dtype=G.dtype, device=DEV)
    n = hlq.hlq_workspace_bytes_mode(N, I, O, B, r, X is None, flags) + extra
    ws = torch.full((n,), 0xFF, dtype=torch.uint8, device=DEV)          # NaN in either type
    hlq.hlq_linear_backward_mode(G, X, Xc, sXc, W, N, I, O, B, r, 9, flags, dX, dW, ws)
    torch.cuda.synchronize()
    return dX, dW


# rows of five steps (the shortest that are padded) to many, ending 16 to 120 bytes into a step; kept coefficients that pad by one
# value, a few and a whole block; 256-tiles, 128-tiles and splits; few and many features
@pytest.mark.parametrize("N,I,O,B,r", [
    (528, 136, 96, 16, 8), (4224, 24, 32, 16, 1), (2112, 264, 160, 32, 4), (1088, 72, 64, 32, 16), (9200, 1160, 624, 16, 8), (12608, 768, 512, 16, 8),
    (1040, 4104, 4112, 16, 16), (8448, 16, 128, 64, 2)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_same_as_from_a_store(N, I, O, B, r, dtype):
    G, X, W = _inputs(N, I, O, dtype)
    Kc = N // B * r
    xc = torch.empty((I, Kc), dtype=torch.bfloat16, device=DEV)
    hlq.hlq_compress_act(X, B, r, xc)
    want = _backward(G, None, xc, None, W, I, B, r, 0)
    got = _backward(G, X, None, None, W, I, B, r, 0)
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    if r >= 4 and Kc % 16 == 0:
        xq, sx = torch.empty((I, Kc), dtype=torch.int8, device=DEV), torch.empty(I, device=DEV)
        ws = torch.empty(hlq.hlq_hla_quantize_workspace_bytes(I), dtype=torch.uint8, device=DEV)
        hlq.hlq_compress_act_int8(X, B, r, 9, xq, sx, ws)
        want = _backward(G, None, xq, sx, W, I, B, r, GWI)
        got = _backward(G, X, None, None, W, I, B, r, GWI)
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    if r >= 8 and Kc % 32 == 0:
        x4 = torch.empty((I, Kc // 2), dtype=torch.uint8, device=DEV)
        hlq.hlq_compress_act_int4(X, B, r, 9, x4, sx, ws)
        low, high = ((x4 << 4).view(torch.int8) >> 4), (x4.view(torch.int8) >> 4)
        want = _backward(G, None, torch.stack((low, high), dim=2).reshape(I, Kc).contiguous(), sx, W, I, B, r, GWI)
        got = _backward(G, None, x4, sx, W, I, B, r, GWI | X4)
        assert all(torch.equal(a, b) for a, b in zip(got, want))


def test_scratch_without_room_for_padding():
    # one byte a code leaves none: the size that a registered workspace needed before rows were padded
    N, I, O, B, r = 528, 136, 96, 16, 8
    flags = hlq.HLQ_FLAG_GX_8BIT
    G, X, W = _inputs(N, I, O, torch.bfloat16)
    want = _backward(G, X, None, None, W, I, B, r, flags)
    pad = sum((rows * 320 * 2 + 255) // 256 * 256 - (rows * 264 * 2 + 255) // 256 * 256 for rows in (O, I))
    got = _backward(G, X, None, None, W, I, B, r, flags, -pad)
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    with pytest.raises(hlq.HlqError):
        _backward(G, X, None, None, W, I, B, r, flags, -pad - 256)


@pytest.mark.parametrize("flags", [0, GWI, hlq.HLQ_FLAG_GX_8BIT])
def test_convolution(flags):
    # 24 x 14 x 14 positions: rows of 2352 values
    geom = hlq.hlq_conv_geom(Nb=24, H=14, W=14, C=16, O=64, kh=3, kw=3, stride_h=1, stride_w=1, pad_h=1, pad_w=1, dil_h=1, dil_w=1)
    N, I, O, B, r = 24 * 196, 144, 64, 16, 8
    G, X, W = _inputs(N, 16, O, torch.float32)[0], _inputs(N, 16, O, torch.float32)[1], _inputs(N, I, O, torch.float32)[2]
    image = X.reshape(24, 14, 14, 16)
    dX, dW = torch.empty_like(image), torch.empty((O, 3, 3, 16), device=DEV)
    ws = torch.full((hlq.hlq_conv_workspace_bytes(geom, B, r, hlq.HLQ_F32, flags),), 0xFF, dtype=torch.uint8, device=DEV)
    hlq.hlq_conv2d_backward(G.reshape(24, 14, 14, O), image, W.reshape(O, 3, 3, 16), geom, B, r, 9, flags, dX, dW, ws)
    cols = torch.nn.functional.unfold(image.permute(0, 3, 1, 2), 3, padding=1)            # [12, 16 * 9, 196]
    cols = cols.reshape(24, 16, 9, 196).permute(0, 3, 2, 1).reshape(N, I).contiguous()
    want = _backward(G, cols, None, None, W, I, B, r, flags)[1]
    assert torch.isfinite(dX).all()
    # the two may split the reduction differently: fp32 sums of N / 2 products
    err = (dW.reshape(O, I) - want).norm() / want.norm()
    assert err < 1e-5, err
