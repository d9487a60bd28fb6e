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


# layers whose plan is a 256-tile dX product beside 128-tiles of dW, for each pair of kinds nine reductions of consecutive step counts: every
# position of the ring's nine units that a last step can end in; edges of rows and columns that fill no tile
FIRST_STEPS = {X8: 25, 0: 22, X8 | GWI: 10, GWI: 15}
LAYERS = {
    X8: [(3168, 936, 512), (3232, 2152, 512), (3392, 784, 640), (3520, 1072, 640), (3616, 784, 768), (3776, 1024, 768), (3968, 904, 896), (4096, 1224, 640),
         (4192, 1168, 640)],
    0: [(2784, 1248, 512), (2944, 1256, 512), (3040, 928, 768), (3136, 776, 688), (3296, 1000, 512), (3392, 800, 640), (3552, 1032, 512), (3648, 792, 512),
        (3744, 856, 640)],
    X8 | GWI: [(2336, 2080, 768), (2784, 1800, 896), (2848, 1872, 768), (3232, 1712, 768), (3360, 1648, 896), (3712, 1664, 768), (3936, 1448, 896),
               (4256, 1448, 768), (4448, 1360, 768)],
    GWI: [(3840, 2368, 3072), (3936, 1344, 3088), (4224, 1168, 2352), (4576, 1032, 2560), (4768, 912, 2832), (4960, 928, 2992), (5184, 656, 2944),
          (5440, 1672, 512), (5792, 640, 512)],
}


@pytest.mark.parametrize("flags", sorted(LAYERS))
@pytest.mark.parametrize("i", range(9))
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_same_bits_as_through_registers(flags, i, dtype):
    B, r = 16, 8
    N, I, O = LAYERS[flags][i]
    steps = FIRST_STEPS[flags] + i
    g = torch.Generator(device=DEV).manual_seed(N)
    G, X, W = (torch.randn(s, generator=g, device=DEV).to(dtype) for s in ((N, O), (N, I), (O, I)))
    # whole reductions, and k splits whose partials come from this body: down to four steps a workgroup, the fewest that take it
    for splits in sorted({1, 2, steps // 5, steps // 4}):
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, splits)
        try:
            plan = hlq.hlq_linear_backward_plan(N, I, O, B, r, flags=flags)
            assert plan[:3] == (256, 128, splits) and plan[5] == (0 if flags & X8 else 2) and plan[6] * (1 if flags & GWI else 2) == 128 * steps
            got = _backward(G, X, W, B, r, flags)
            hlq.hlq_set_option(hlq.HLQ_OPT_DIRECT_TO_LDS, 0)
            want = _backward(G, X, W, B, r, flags)
        finally:
            hlq.hlq_set_option(hlq.HLQ_OPT_DIRECT_TO_LDS, 1)
            hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, 0)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), splits
