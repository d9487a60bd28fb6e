"""The whole path keeps the 4-bit codes of the g_x list in the layout that widens to 6-bit floats.
Their product is exact, so dX is the same bit for bit as with one int8 a code (HLQ_FLAG_GX_UNPACKED), which the other
tests hold to the oracle."""
import pytest
import torch

import paper_2406_15102_amd as hlq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
UNPACKED = hlq.HLQ_FLAG_GX_UNPACKED


def _inputs(N, I, O, dtype, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    G = torch.randn((N, O), generator=g, device=DEV) * torch.exp(torch.randn((N, 1), generator=g, device=DEV)) * 1e-3
    X = torch.randn((N, I), generator=g, device=DEV)
    W = torch.randn((O, I), generator=g, device=DEV) * 0.02
    return G.to(dtype), X.to(dtype), W.to(dtype)


def _run(G, X, W, B, r, flags, want_dw=True, cached=False):
    N, O, I = G.shape[0], G.shape[1], W.shape[1]
    dX = torch.full((N, I), 7.0, dtype=G.dtype, device=DEV)
    dW = torch.full((O, I), 7.0, dtype=G.dtype, device=DEV) if want_dw else None
    ws = torch.full((hlq.hlq_workspace_bytes_mode(N, I, O, B, r, False, flags),), 255, dtype=torch.uint8, device=DEV)
    if cached:
        bits = hlq.hlq_weight_code_bits(O, flags)
        Wc = torch.empty((I, O // 2 if bits & 0x1FF == hlq.HLQ_BITS_4_PACKED else O), dtype=torch.int8, device=DEV)
        sW = torch.empty(I, dtype=torch.float32, device=DEV)
        hlq.hlq_quantize_w(W, B, 5, Wc, sW, torch.empty(hlq.hlq_quantize_w_workspace_bytes(O, I), dtype=torch.uint8, device=DEV), None, bits)
        hlq.hlq_linear_backward_cached(G, X if want_dw else None, None, None, Wc, sW, N, I, O, B, r, 5, flags, dX, dW, ws)
    else:
        hlq.hlq_linear_backward_mode(G, X if want_dw else None, None, None, W, N, I, O, B, r, 5, flags, dX, dW, ws)
    torch.cuda.synchronize()
    return dX, dW


def _same(a, b):
    return torch.equal(torch.nan_to_num(a, nan=1e30), torch.nan_to_num(b, nan=1e30))


# rows of codes of one to many steps, whole and padded (208, 240, 400: half a group of 32 codes at the end), every split of a
# row over lanes (4 to 256 lanes, 1024 for the longest), token and feature counts that fill no tile
SHAPES = [(320, 136, 240, 16), (64, 24, 208, 16), (400, 264, 400, 16), (1024, 520, 768, 32), (640, 72, 1024, 64), (528, 1032, 3072, 16),
          (4096, 1000, 1408, 32), (512, 2048, 5632, 64), (256, 512, 6160, 16), (272, 96, 11008, 16), (128, 64, 16384 + 64, 64),
          (64, 16, 65536, 64), (2304, 4104, 2064, 16), (8192, 768, 512, 32), (16, 8, 256, 16)]


@pytest.mark.parametrize("N,I,O,B", SHAPES)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_same_bits_as_bytes(N, I, O, B, dtype):
    G, X, W = _inputs(N, I, O, dtype, N + I + O)
    G[N // 2] = 0
    W[:, 3] = 0
    for flags, want_dw in ((0, True), (0, False), (hlq.HLQ_FLAG_GW_INT8, True), (hlq.HLQ_FLAG_ROUND_MANTISSA, True)):
        if flags & hlq.HLQ_FLAG_GW_INT8 and N // B * 8 % 16:
            continue
        if N // B * 8 % 8:
            continue
        a, _ = _run(G, X, W, B, 8, flags, want_dw)
        b, _ = _run(G, X, W, B, 8, flags | UNPACKED, want_dw)
        assert _same(a, b), (flags, want_dw)
        assert float(a.float().abs().max()) > 0


@pytest.mark.parametrize("N,I,O,B", [(400, 264, 400, 16), (1024, 520, 768, 32), (4096, 4104, 1408, 32), (256, 512, 6160, 16), (128, 64, 16448, 64)])
@pytest.mark.parametrize("flags", [0, hlq.HLQ_FLAG_GW_INT8])
def test_weight_codes_handed_over(N, I, O, B, flags):
    G, X, W = _inputs(N, I, O, torch.bfloat16, 3 * N + I)
    a, _ = _run(G, X, W, B, 16, flags)
    for mix in (1, 0):
        try:
            hlq.hlq_set_option(hlq.HLQ_OPT_FRONT_INTERLEAVE, mix)
            for want_dw in (True, False):
                b, _ = _run(G, X, W, B, 16, flags, want_dw, cached=True)
                assert torch.equal(a, b)
        finally:
            hlq.hlq_set_option(hlq.HLQ_OPT_FRONT_INTERLEAVE, 1)


@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("gw", [0, hlq.HLQ_FLAG_GW_INT8])
def test_either_tile(tile, splits, gw):
    # 3 and 13 steps of codes, a dW product of whole and of ragged steps
    for N, I, O, B in ((2048 + 64, 392, 656, 16), (1024, 1000, 3264, 32)):
        G, X, W = _inputs(N, I, O, torch.bfloat16, 11)
        want, _ = _run(G, X, W, B, 16, gw | UNPACKED)
        try:
            hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_TILE, tile)
            hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, splits)
            for f in (0, hlq.HLQ_FLAG_SEPARATE_PRODUCTS):
                dX, dW = _run(G, X, W, B, 16, gw | f)
                assert torch.equal(dX, want)
        finally:
            hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_TILE, 0)
            hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, 0)


@pytest.mark.parametrize("B", [16, 32, 64])
def test_codes_that_are_none(B):
    """Rows and columns whose largest value is below 7 / FLT_MAX (an infinite reciprocal scale), infinities and NaN: the codes
    are those that an int8 of them has."""
    N, I, O = 192, 72, 448
    G, X, W = _inputs(N, I, O, torch.float32, 17)
    G[5] *= 1e-36
    G[6] = 0
    G[6, 40] = 1e-39
    G[7, 3] = float("nan")
    G[8, 100] = float("inf")
    G[9] *= 1e38
    W[:, 2] *= 1e-37
    W[33, 4] = float("nan")
    W[200, 9] = float("-inf")
    a, _ = _run(G, X, W, B, 8, 0, want_dw=False)
    b, _ = _run(G, X, W, B, 8, UNPACKED, want_dw=False)
    assert _same(a, b)
    for c in (0, hlq.HLQ_FLAG_GX_UNPACKED):
        d, _ = _run(G, X, W, B, 8, c, want_dw=False, cached=True)
        assert _same(a, d)


def test_longest_sums_are_exact():
    """All codes at their largest: 49 K = 3.2 million, every partial sum a whole number."""
    N, I, O, B = 64, 16, 65536, 16
    W = torch.zeros((O, I), dtype=torch.float32, device=DEV)
    G = torch.zeros((N, O), dtype=torch.float32, device=DEV)
    G[:, ::16] = torch.where(torch.rand((N, 1), device=DEV) < 0.5, -1.0, 1.0)    # one value a block: B equal coefficients
    W[::16, :] = 1.0
    W[16 * 7:16 * 9:16, 1] = -1.0
    X = torch.zeros((N, I), device=DEV)
    a, _ = _run(G, X, W, B, 8, 0, want_dw=False)
    b, _ = _run(G, X, W, B, 8, UNPACKED, want_dw=False)
    assert torch.equal(a, b)
    # 65536 / 16 of +-1, up to the rounding of the two scales 1/7 and of three products: 5 * 2^-24
    assert abs(float(a.abs().max()) - 4096.0) <= 4096.0 * 5 * 2.0 ** -24
