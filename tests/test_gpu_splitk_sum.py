"""The reduction of split-k partials: rounds of four loads up to four splits, of eight beyond, the last round's spare loads not
added.  Integer partials, so the sums are exact; values in bf16 products are whole and small enough to be exact too."""
import pytest
import torch

import paper_2406_15102_amd as hlq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("splits", [2, 3, 4, 5, 7, 8, 9, 12, 15, 16])
@pytest.mark.parametrize("M,N", [(128, 132), (72, 20)])
def test_every_number_of_splits(splits, M, N):
    K = 4096
    g = torch.Generator(device=DEV).manual_seed(splits)
    A = torch.randint(-7, 8, (M, K), generator=g, device=DEV, dtype=torch.int8)
    Bm = torch.randint(-7, 8, (N, K), generator=g, device=DEV, dtype=torch.int8)
    want = (A.double() @ Bm.double().t()).float()                       # below 2^24: exact in fp32 whatever the order
    ws = torch.full((16 * M * N * 4,), 0xFF, dtype=torch.uint8, device=DEV)
    try:
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, splits)
        C = torch.empty((M, N), device=DEV)
        hlq.hlq_int8_gemm_nt(A, Bm, None, None, 1.0, C, None, ws)
        D = torch.empty((M, N), device=DEV)
        hlq.hlq_bf16_gemm_nt(A.bfloat16(), Bm.bfloat16(), 1.0, D, ws)
        torch.cuda.synchronize()
    finally:
        hlq.hlq_set_option(hlq.HLQ_OPT_PLAN_SPLITS, 0)
    assert torch.equal(C, want) and torch.equal(D, want)
