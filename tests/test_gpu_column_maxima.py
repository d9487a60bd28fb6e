"""Integer g_w list: where every tensor of the call has at most 4096 rows, and the scratch room, the column maxima are
left as tables that the second pass folds, otherwise they are merged by atomics; a 4-bit store is widened beside the
first passes; an image is projected there too.  Each way, the pass gives the bits that the stage entry points give (which merge by atomics)."""
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
    (4096 + 64, 136, 4096, 64, 32),     # by atomics: too many tokens
    (512, 72, 4096 + 32, 32, 16),       # too many out-features
    (4096 + 32, 40, 4096 + 32, 32, 32), # both
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


# The same equality over the forms that the tests above leave out: element type, kind of the g_x codes, basis, weight codes
# handed over, one gradient alone, the quantiser's workgroups in their own range.
CODES8, UNPACKED, SEQ = hlq.HLQ_FLAG_GX_8BIT, hlq.HLQ_FLAG_GX_UNPACKED, hlq.HLQ_FLAG_GW_SEQUENCY
SHAPES = [
    (1024, 72, 1056, 32, 16),           # every tensor with a table, the last row of the weight's partly filled
    (4096 + 64, 136, 4096, 64, 32),     # too many tokens for a table: one for the weight only where it is alone
    (512, 72, 4096 + 32, 32, 16),       # too many out-features: a table for the tokens only without a pass over the weight
    (4096 + 32, 40, 4096 + 32, 32, 32), # all by atomics
    (4096, 8192, 320, 16, 8),           # few enough reads of the tables (2.21 M)
    (4096, 8192, 640, 16, 8),           # too many (2.33 M): all by atomics
]


def _stages(G, X, W, B, r, seed, flags):
    """The operands of both products from the stage entry points: (Gq, sG, Wq, sW, bits, Gh, sGh, Xh, sXh)."""
    (N, O), I = G.shape, X.shape[1]
    Kc = N // B * r
    ws = _empty(1 << 20, torch.uint8)
    bits = hlq.hlq_weight_code_bits(O, flags)
    width = O // 2 if bits == hlq.HLQ_BITS_4_PACKED else O
    Gq, sG, Wq, sW = _empty((N, width), torch.int8), _empty(N, torch.float32), _empty((I, width), torch.int8), _empty(I, torch.float32)
    hlq.hlq_quantize_g(G, B, seed, Gq, sG, None, bits)
    hlq.hlq_quantize_w(W, B, seed, Wq, sW, ws, None, bits)
    basis = 1 if flags & SEQ else 0
    Gh, sGh, Xh, sXh = _empty((O, Kc), torch.int8), _empty(O, torch.float32), _empty((I, Kc), torch.int8), _empty(I, torch.float32)
    hlq.hlq_hla_quantize_basis(G, B, r, basis, seed, 3, Gh, sGh, ws)
    hlq.hlq_hla_quantize_basis(X, B, r, basis, seed, 2, Xh, sXh, ws)
    return Gq, sG, Wq, sW, bits, Gh, sGh, Xh, sXh


def _tensors(N, d_in, d_out, dtype):
    return (dev(rand_tensor((N, d_out), dtype, 1, 1e-3, 0.7)), dev(rand_tensor((N, d_in), dtype, 3, 1.0, 0.5)),
            dev(rand_tensor((d_out, d_in), dtype, 2, 0.02)))


def _filled(n):
    return torch.full((n,), 0xFF, dtype=torch.uint8, device=DEV)


@pytest.mark.parametrize("N,d_in,d_out,B,r", SHAPES)
@pytest.mark.parametrize("form", ["f32", "8bit", "unpacked", "sequency", "codes", "codes_int8_store", "dx", "dw"])
def test_forms_equal_their_stages(N, d_in, d_out, B, r, form):
    G, X, W = _tensors(N, d_in, d_out, torch.float32 if form == "f32" else torch.bfloat16)
    flags = GWI | {"8bit": CODES8, "unpacked": UNPACKED, "sequency": SEQ}.get(form, 0)
    ops = _stages(G, X, W, B, r, 9, flags)
    dX, dW = _empty((N, d_in), G.dtype), _empty((d_out, d_in), G.dtype)
    hlq.hlq_backward_products(*ops, B, dX, dW, None)
    Wq, sW, Xh, sXh = ops[2], ops[3], ops[7], ops[8]
    store = form == "codes_int8_store"
    a = None if form == "dw" else torch.zeros_like(dX)
    b = None if form == "dx" else torch.zeros_like(dW)
    x = (None, Xh, sXh) if store else (X, None, None)
    ws = _filled(hlq.hlq_workspace_bytes_mode(N, d_in, d_out, B, r, store, flags))
    if form.startswith("codes"):
        hlq.hlq_linear_backward_cached(G, *x, Wq, sW, N, d_in, d_out, B, r, 9, flags, a, b, ws)
    else:
        hlq.hlq_linear_backward_mode(G, *x, W, N, d_in, d_out, B, r, 9, flags, a, b, ws)
    assert a is None or torch.equal(a, dX)
    assert b is None or torch.equal(b, dW)
    assert float(dX.float().abs().max()) > 0 and float(dW.float().abs().max()) > 0


@pytest.mark.parametrize("N,d_in,d_out,B,r", SHAPES)
def test_int4_store_without_the_turns(N, d_in, d_out, B, r):
    G, X, W = _tensors(N, d_in, d_out, torch.bfloat16)
    dX, dW, Xc, sXc = _by_stages(G, X, W, B, r, 9, "int4")
    ws = _filled(hlq.hlq_workspace_bytes_mode(N, d_in, d_out, B, r, True, GWI | X4))
    a, b = torch.zeros_like(dX), torch.zeros_like(dW)
    try:
        hlq.hlq_set_option(hlq.HLQ_OPT_FRONT_INTERLEAVE, 0)
        hlq.hlq_linear_backward_mode(G, None, Xc, sXc, W, N, d_in, d_out, B, r, 9, GWI | X4, a, b, ws)
    finally:
        hlq.hlq_set_option(hlq.HLQ_OPT_FRONT_INTERLEAVE, 1)
    assert torch.equal(a, dX) and torch.equal(b, dW)


@pytest.mark.parametrize("H,C,stride,dtype", [(16, 24, 1, torch.bfloat16), (32, 40, 2, torch.float32), (36, 16, 1, torch.bfloat16)])
def test_image_gradient_equals_the_folded_columns(H, C, stride, dtype):
    Nb, O, k, B, r = 4, 48, 3, 16, 8
    geom = hlq.hlq_conv_geom(Nb=Nb, H=H, W=H, C=C, O=O, kh=k, kw=k, stride_h=stride, stride_w=stride, pad_h=1, pad_w=1, dil_h=1, dil_w=1)
    Ho, Wo, N, I = hlq.hlq_conv_sizes(geom)
    X = dev(rand_tensor((Nb, H, H, C), dtype, 5, 1.0))
    W, G = dev(rand_tensor((O, k, k, C), dtype, 6, 0.02)), dev(rand_tensor((Nb, Ho, Wo, O), dtype, 7, 1e-3))
    cols = _empty((N, I), dtype)
    hlq.hlq_im2col(X, geom, cols)
    dX, dW, want = torch.zeros_like(X), torch.empty_like(W), torch.empty_like(X)
    hlq.hlq_conv2d_backward(G, X, W, geom, B, r, 9, GWI, dX, dW, None)
    cols_grad, _, _, _ = _by_stages(G.reshape(N, O), cols, W.reshape(O, I), B, r, 9, None)
    hlq.hlq_col2im(cols_grad, geom, want)
    assert torch.equal(dX, want)
    assert float(dX.float().abs().max()) > 0


# Scratch sized for a longer problem, whose maxima have no table, holds a shorter one: the tables are left out where the
# scratch has no room for them.  The bytes behind it stay as they are.
@pytest.mark.parametrize("longer,shorter", [
    ((4112, 96, 768, 16, 16), (4096, 96, 768, 16, 16)),          # tokens: 4096 have a table, 4112 none
    ((256, 256, 4112, 16, 16), (256, 256, 4096, 16, 16)),        # out-features
    ((4128, 24, 4128, 32, 32), (4096, 24, 4096, 32, 32)),        # both
])
def test_scratch_of_a_longer_problem(longer, shorter):
    room, need = hlq.hlq_workspace_bytes_mode(*longer[:5], False, GWI), hlq.hlq_workspace_bytes_mode(*shorter[:5], False, GWI)
    assert room < need                   # what the case is about
    N, d_in, d_out, B, r = shorter
    G, X, W = _tensors(N, d_in, d_out, torch.bfloat16)
    dX, dW, _, _ = _by_stages(G, X, W, B, r, 9, None)
    memory = _filled(room + (1 << 20))
    a, b = torch.zeros_like(dX), torch.zeros_like(dW)
    hlq.hlq_linear_backward_mode(G, X, None, None, W, N, d_in, d_out, B, r, 9, GWI, a, b, memory[:room])
    assert torch.equal(a, dX) and torch.equal(b, dW)
    assert bool((memory[room:] == 0xFF).all())
    a.zero_(), b.zero_(), memory.fill_(0xFF)
    try:
        hlq.hlq_set_workspace(memory[:room])
        hlq.hlq_linear_backward_mode(G, X, None, None, W, N, d_in, d_out, B, r, 9, GWI, a, b, None)
        torch.cuda.synchronize()
    finally:
        hlq.hlq_set_workspace(None)
    assert torch.equal(a, dX) and torch.equal(b, dW)
    assert bool((memory[room:] == 0xFF).all())


def test_scratch_of_a_longer_convolution():
    B, r, flags = 16, 16, GWI

    def geom(Nb, C=8, O=1024):
        return hlq.hlq_conv_geom(Nb=Nb, H=4, W=4, C=C, O=O, kh=3, kw=3, stride_h=1, stride_w=1, pad_h=1, pad_w=1, dil_h=1, dil_w=1)
    room, need = (hlq.hlq_conv_workspace_bytes(geom(Nb), B, r, hlq.HLQ_BF16, flags) for Nb in (257, 256))
    assert room < need
    X = dev(rand_tensor((256, 4, 4, 8), torch.bfloat16, 5, 1.0))
    W, G = dev(rand_tensor((1024, 3, 3, 8), torch.bfloat16, 6, 0.02)), dev(rand_tensor((256, 4, 4, 1024), torch.bfloat16, 7, 1e-3))
    memory = _filled(need)
    out = []
    for n in (need, room):
        dX, dW = torch.zeros_like(X), torch.zeros_like(W)
        memory.fill_(0xFF)
        hlq.hlq_conv2d_backward(G, X, W, geom(256), B, r, 9, flags, dX, dW, memory[:n])
        out.append((dX, dW))
    assert bool((memory[room:] == 0xFF).all())
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert float(out[0][1].float().abs().max()) > 0
