"""Weight codes that are handed over stay nibbles or bytes where bringing them into the layout of the 6-bit floats would not pay
(few tokens, a weight that no cache holds): the same bits as the call that quantises the weight itself, on either side of the rule."""
import pytest
import torch

import paper_2406_15102_amd as hlq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
B, r, SEED = 16, 8, 5
GWI = hlq.HLQ_FLAG_GW_INT8


# either side of the rule's lines: 2^25 codes and more, 1024 tokens and more, 2048 with the integer list, 480 and 512 for dX alone, 2^27 codes;
# as nibbles and as bytes (8208 out-features)
@pytest.mark.parametrize("N,I,O", [(1024, 8192, 8192), (1056, 8200, 8192), (288, 8200, 8208), (2048, 8200, 4128), (480, 4104, 8192), (512, 4104, 8192), (288, 4096, 8192), (288, 8200, 16416)])
@pytest.mark.parametrize("flags", [0, GWI])
def test_same_bits_as_quantised_here(N, I, O, flags):
    g = torch.Generator(device=DEV).manual_seed(N + I)
    G, X, W = (torch.randn(s, generator=g, device=DEV).to(torch.bfloat16) for s in ((N, O), (N, I), (O, I)))
    bits = hlq.hlq_weight_code_bits(O, flags)
    Wc = torch.empty((I, O // 2 if bits == hlq.HLQ_BITS_4_PACKED else O), dtype=torch.int8, device=DEV)
    sW = torch.empty(I, dtype=torch.float32, device=DEV)
    hlq.hlq_quantize_w(W, B, SEED, Wc, sW, torch.empty(hlq.hlq_quantize_w_workspace_bytes(O, I), dtype=torch.uint8, device=DEV), None, bits)
    want = torch.empty((N, I), dtype=torch.bfloat16, device=DEV)
    dW0 = torch.empty((O, I), dtype=torch.bfloat16, device=DEV)
    ws = torch.full((hlq.hlq_workspace_bytes_mode(N, I, O, B, r, False, flags),), 255, dtype=torch.uint8, device=DEV)
    hlq.hlq_linear_backward_mode(G, X, None, None, W, N, I, O, B, r, SEED, flags, want, dW0, ws)
    for dw in (True, False):
        dX = torch.full_like(want, 7.0)
        dW = torch.full_like(dW0, 7.0) if dw else None
        ws.fill_(255)
        hlq.hlq_linear_backward_cached(G, X if dw else None, None, None, Wc, sW, N, I, O, B, r, SEED, flags, dX, dW, ws)
        torch.cuda.synchronize()
        assert torch.equal(dX, want)
        # dW: the same operands, the sums of at most 1024 products in another order where the tiles are others
        if dw:
            assert (dW.float() - dW0.float()).norm() <= 2.0 ** -8 * dW0.float().norm()
