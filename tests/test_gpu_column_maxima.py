"""Integer g_w list: up to 4096 rows the column maxima are left as a table that the second pass folds, beyond they
are merged by atomics, tensor by tensor; a 4-bit store is widened beside the first passes; an image is projected
there too.  Each way, the pass gives the bits that the stage entry points give (which merge by atomics)."""
import pytest
import torch

import paper_2406_15102_amd as hlq
from test_gpu_parity import dev, rand_tensor

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GWI, X4 = hlq.HLQ_FLAG_GW_INT8, hlq.HLQ_FLAG_XC_INT4


def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV)


def _by_stages(G, X, W, B, r, seed, store):
    """-> (dX, dW, Xc, sXc); Xc as the int8 or 4-bit store."""
    (N, O), I = G.shape, X.shape[1]
    Kc = N // B * r
    ws = _empty(1 << 20, torch.uint8)
    bits = hlq.hlq_weight_code_bits(O, GWI)
    width = O // 2 if bits == hlq.HLQ_BITS_4_PACKED else O
    Gq, sG, Wq, sW = _empty((N, width), torch.int8), _empty(N, torch.float32), _empty((I, width), torch.int8), _empty(I, torch.float32)
    hlq.hlq_quantize_g(G, B, seed, Gq, sG, None, bits)
    hlq.hlq_quantize_w(W, B, seed, Wq, sW, ws, None, bits)
    Gh, sGh, Xc, sXc = _empty((O, Kc), torch.int8), _empty(O, torch.float32), _empty((I, Kc), torch.int8), _empty(I, torch.float32)
    hlq.hlq_hla_quantize(G, B, r, seed, 3, Gh, sGh, ws)
    Xh = Xc
    if store == "int4":
        Xc = _empty((I, Kc // 2), torch.uint8)
        hlq.hlq_compress_act_int4(X, B, r, seed, Xc, sXc, ws)
        n = torch.stack((Xc & 15, Xc >> 4), dim=2).to(torch.int16)
        Xh = torch.where(n > 7, n - 16, n).to(torch.int8).reshape(I, Kc).contiguous()
    else:
        hlq.hlq_hla_quantize(X, B, r, seed, 2, Xc, sXc, ws)
    dX, dW = _empty((N, I), G.dtype), _empty((O, I), G.dtype)
    hlq.hlq_backward_products(Gq, sG, Wq, sW, bits, Gh, sGh, Xh, sXc, B, dX, dW, None)
    return dX, dW, Xc, sXc


@pytest.mark.parametrize("N,d_in,d_out,B,r", [
    (64, 64, 16, 16, 8),                # one row of workgroups
    (4096, 136, 48, 16, 8),             # the largest table of tokens
    (4096 + 64, 136, 4096, 64, 32),     # tokens by atomics, the weight's out-features at the largest table
    (512, 72, 4096 + 32, 32, 16),       # the other way round
    (4096 + 32, 40, 4096 + 32, 32, 32), # all by atomics
])
@pytest.mark.parametrize("store", [None, "int8", "int4"])
def test_pass_equals_its_stages(N, d_in, d_out, B, r, store):
    G, W = dev(rand_tensor((N, d_out), torch.bfloat16, 1, 1e-3, 0.7)), dev(rand_tensor((d_out, d_in), torch.bfloat16, 2, 0.02))
    X = dev(rand_tensor((N, d_in), torch.bfloat16, 3, 1.0, 0.5))
    dX, dW, Xc, sXc = _by_stages(G, X, W, B, r, 9, store)
    flags = GWI | (X4 if store == "int4" else 0)
    ws = torch.full((hlq.hlq_workspace_bytes_mode(N, d_in, d_out, B, r, store is not None, flags),), 0xFF, dtype=torch.uint8, device=DEV)
    a, b = _empty((N, d_in), G.dtype), _empty((d_out, d_in), G.dtype)
    hlq.hlq_linear_backward_mode(G, None if store else X, Xc if store else None, sXc if store else None, W, N, d_in, d_out, B, r, 9,
                                 flags, a, b, ws)
    assert torch.equal(a, dX) and torch.equal(b, dW)
    assert float(dW.float().abs().max()) > 0


@pytest.mark.parametrize("H,C,stride,dtype", [(16, 24, 1, torch.bfloat16), (32, 40, 2, torch.float32), (36, 16, 1, torch.bfloat16)])
def test_image_equals_its_column_matrix(H, C, stride, dtype):
    Nb, O, k, B, r = 4, 48, 3, 16, 8
    geom = hlq.hlq_conv_geom(Nb=Nb, H=H, W=H, C=C, O=O, kh=k, kw=k, stride_h=stride, stride_w=stride, pad_h=1, pad_w=1, dil_h=1, dil_w=1)
    Ho, Wo, N, I = hlq.hlq_conv_sizes(geom)
    X = dev(rand_tensor((Nb, H, H, C), dtype, 5, 1.0))
    W, G = dev(rand_tensor((O, k, k, C), dtype, 6, 0.02)), dev(rand_tensor((Nb, Ho, Wo, O), dtype, 7, 1e-3))
    cols = _empty((N, I), dtype)
    hlq.hlq_im2col(X, geom, cols)
    dX, dW = torch.empty_like(X), torch.empty_like(W)
    hlq.hlq_conv2d_backward(G, X, W, geom, B, r, 9, GWI, dX, dW, None)
    _, want, _, _ = _by_stages(G.reshape(N, O), cols, W.reshape(O, I), B, r, 9, None)
    assert torch.equal(dW.reshape(O, I), want)
