"""Both products of a pass on 128 x 128 tiles whose operands go straight into LDS (k steps that are not whole
included), at the smallest sizes that take that form: work for two tiles a compute unit, two whole steps a workgroup.  Held to the
bits of the register-staged form, and to sums of the same operands in 64 bits."""
import pytest
import torch

import paper_2406_15102_amd as hlq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _codes(rows, K, bits, gen):
    if bits == hlq.HLQ_BITS_8:
        q = torch.randint(-127, 128, (rows, K), generator=gen, dtype=torch.int16)
    else:
        q = torch.randint(-7, 8, (rows, K), generator=gen, dtype=torch.int16)
    store = ((q[:, 0::2] & 15) | ((q[:, 1::2] & 15) << 4)).to(torch.uint8).view(torch.int8) if bits == hlq.HLQ_BITS_4_PACKED else q.to(torch.int8)
    return q.to(torch.float64).to(DEV), store.contiguous().to(DEV)


P4, I8 = hlq.HLQ_BITS_4_PACKED, hlq.HLQ_BITS_8


@pytest.mark.parametrize("N,d_in,d_out,Kc,bits,gw_int8,f32,splits", [
    (8192, 1152, 1024, 256, P4, False, False, 1),           # whole steps and tiles throughout
    (8184, 1032, 1024, 256 + 8, P4, False, False, 1),       # 16 bytes of a last step, tiles over both edges
    (8184, 1028, 1024, 256 + 32, P4, False, True, 1),       # half a step; fp32; rows of C not 16 bytes of bf16
    (8184, 1028, 1024 + 32, 256 + 40, P4, False, False, 1),     # 16 bytes of packed codes
    (8192, 1152, 512 + 224, 128 + 56, P4, False, True, 1),  # all but 16 bytes, two whole steps
    (8192, 1152, 512 + 96, 512 + 120, P4, False, False, 3),     # split reduction, the last part with the ragged step
    (8192, 1152, 512 + 160, 1024 + 8, P4, False, True, 8),  # two whole steps a part
    (8192, 1152, 256 + 16, 128 + 24, I8, False, False, 1),  # one int8 a code
    (8200, 1160, 512 + 112, 256 + 64, I8, False, True, 2),
    (8192, 1152, 1024 + 64, 256 + 16, P4, True, False, 1),  # integer projections: int8 for the g_w product
    (8192, 1152, 256 + 80, 512 + 112, I8, True, True, 2),
])
def test_128_tiles_straight_into_lds(N, d_in, d_out, Kc, bits, gw_int8, f32, splits):
    gen = torch.Generator().manual_seed(N + d_in + d_out + Kc)
    G, Gq = _codes(N, d_out, bits, gen)
    W, Wq = _codes(d_in, d_out, bits, gen)
    sG, sW = torch.rand(N, generator=gen).to(DEV), torch.rand(d_in, generator=gen).to(DEV)
    if gw_int8:
        Gh64, Gh = _codes(d_out, Kc, I8, gen)
        Xh64, Xh = _codes(d_in, Kc, I8, gen)
        sGh, sXh = torch.rand(d_out, generator=gen).to(DEV), torch.rand(d_in, generator=gen).to(DEV)
    else:
        Gh, Xh = (torch.randn((n, Kc), generator=gen).to(torch.bfloat16).to(DEV) for n in (d_out, d_in))
        Gh64, Xh64, sGh, sXh = Gh.double(), Xh.double(), None, None
    dt = torch.float32 if f32 else torch.bfloat16
    ws = torch.zeros(64 << 20, dtype=torch.uint8, device=DEV)
    got = []
    try:
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_TILE, 128)
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, splits)
        for direct in (0, 1):
            hlq.hlq_set_option(hlq.HLQ_OPT_DIRECT_TO_LDS, direct)
            dX, dW = torch.zeros((N, d_in), dtype=dt, device=DEV), torch.zeros((d_out, d_in), dtype=dt, device=DEV)
            hlq.hlq_backward_products(Gq, sG, Wq, sW, bits, Gh, sGh, Xh, sXh, 16, dX, dW, ws)
            torch.cuda.synchronize()
            got.append((dX, dW))
    finally:
        hlq.hlq_set_option(hlq.HLQ_OPT_DIRECT_TO_LDS, 1)
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, 0)
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_TILE, 0)
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    dX, dW = got[1]
    rX = (G @ W.T) * sG.double()[:, None] * sW.double() / 16
    rW = Gh64 @ Xh64.T / 16
    if gw_int8:
        rW = rW * sGh.double()[:, None] * sXh.double()
    # exact integer sums, three roundings to fp32 and one to the type (8 bits of significand in bf16: half a unit in the
    # last place is up to 2^-8 of the value); the bf16 products sum Kc terms in fp32
    eps = 2.0 ** -24 if f32 else 2.0 ** -8
    assert torch.all((dX.double() - rX).abs() <= rX.abs() * (eps + 2.0 ** -22))
    bound = rW.abs() * (eps + 2.0 ** -22)
    if not gw_int8:
        bound = bound + (Gh64.abs() @ Xh64.abs().T) / 16 * Kc * 2.0 ** -24
    assert torch.all((dW.double() - rW).abs() <= bound)


def test_128_tiles_infinity_past_a_row_end():
    """A ragged step's lanes past the end of a row multiply nothing: values of the next row that are not finite stay
    in their own row and column of dW."""
    gen = torch.Generator().manual_seed(5)
    N, d_in, d_out, Kc = 8192, 1152, 1024, 256 + 8
    _, Gq = _codes(N, d_out, P4, gen)
    _, Wq = _codes(d_in, d_out, P4, gen)
    sG, sW = torch.rand(N, generator=gen).to(DEV), torch.rand(d_in, generator=gen).to(DEV)
    Gh, Xh = (torch.randn((n, Kc), generator=gen).to(torch.bfloat16).to(DEV) for n in (d_out, d_in))
    Gh[5] = float("inf")
    Xh[7] = float("nan")
    dX, dW = torch.zeros((N, d_in), device=DEV), torch.zeros((d_out, d_in), device=DEV)
    try:
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_TILE, 128)
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, 1)
        hlq.hlq_backward_products(Gq, sG, Wq, sW, P4, Gh, None, Xh, None, 16, dX, dW, None)
        torch.cuda.synchronize()
    finally:
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, 0)
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_TILE, 0)
    finite = torch.isfinite(dW)
    assert not finite[5].any() and not finite[:, 7].any()
    finite[5], finite[:, 7] = True, True
    assert finite.all()
