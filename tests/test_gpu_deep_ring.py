"""128-tiles of the dW product beside 256-tiles of the dX product: the ring of LDS units that is four steps ahead instead of two.
Same steps in the same order, so dW is the same bit for bit as with its operands staged through registers."""
import pytest
import torch

import paper_2406_15102_amd as hlq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GWI, X8 = hlq.HLQ_FLAG_GW_INT8, hlq.HLQ_FLAG_GX_8BIT


def _backward(G, X, W, B, r, flags):
    N, O, I = G.shape[0], G.shape[1], W.shape[1]
    dX, dW = torch.empty((N, I), dtype=G.dtype, device=DEV), torch.empty((O, I), dtype=G.dtype, device=DEV)
    ws = torch.full((hlq.hlq_workspace_bytes_mode(N, I, O, B, r, False, flags),), 0xFF, dtype=torch.uint8, device=DEV)
    hlq.hlq_linear_backward_mode(G, X, None, None, W, N, I, O, B, r, 3, flags, dX, dW, ws)
    torch.cuda.synchronize()
    return dX, dW


# plans of a 256-tile dX product and an unsplit 128-tile dW product of 23 to 64 steps (every position of the ring's nine units a
# last step can end in), edges of rows and columns that fill no tile; with int8 projections half the steps
@pytest.mark.parametrize("N,I,O", [(2848, 2040, 2304), (3104, 1216, 1920), (3840, 1856, 1152), (4352, 2240, 3072), (4640, 1512, 1280), (4896, 1616, 896),
                                   (5376, 1304, 1024), (8192, 2144, 512), (6144, 736, 2944)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_same_bits_as_through_registers(N, I, O, dtype):
    B, r = 16, 8
    assert tuple(hlq.hlq_backward_products_plan(N, I, O, N // B * r, hlq.HLQ_BITS_8, False, 1 << 28)[:3]) == (256, 128, 1)
    g = torch.Generator(device=DEV).manual_seed(N)
    G, X, W = (torch.randn(s, generator=g, device=DEV).to(dtype) for s in ((N, O), (N, I), (O, I)))
    for flags in (X8, 0, X8 | GWI):
        if flags & GWI and N // B * r % 16:
            continue
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, 1)
        try:
            got = _backward(G, X, W, B, r, flags)
            hlq.hlq_set_option(hlq.HLQ_OPT_DIRECT_TO_LDS, 0)
            want = _backward(G, X, W, B, r, flags)
        finally:
            hlq.hlq_set_option(hlq.HLQ_OPT_DIRECT_TO_LDS, 1)
            hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, 0)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
