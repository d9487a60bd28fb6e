"""The projection read through an image at blocks of 32 and 64 rows steps byte offsets from position to position and
leaves taps outside the image to the range check of the load: the same bits as the projection of the stored column
matrix, on either side of the size beyond which the images of a wavefront are not addressed in 32 bits."""
import pytest
import torch

import paper_2406_15102_amd as hlq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# Nb, H, W, C, k, stride, pad, dilation: rows and images that end inside a block, strides past the kernel, taps that meet
# no pixel, one output position per image (a block of rows is B images) small enough for 32 bits and too large
CASES = [(2, 7, 9, 8, 3, 1, 1, 1), (4, 16, 8, 8, 5, 2, 2, 1), (8, 5, 5, 24, 3, 3, 4, 2), (16, 9, 4, 16, 2, 1, 0, 3), (64, 3, 3, 8, 3, 1, 0, 1),
         (64, 704, 704, 8, 3, 1024, 1, 1), (64, 720, 720, 8, 3, 1024, 1, 1)]


@pytest.mark.parametrize("B", [32, 64])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("c", CASES)
def test_projection_through_the_image_equals_that_of_the_columns(c, dtype, B):
    Nb, H, W, C, k, s, p, d = c
    if H > 64 and dtype == torch.float32:
        Nb = 64 if B == 64 else 32
    Ho, Wo = (H + 2 * p - d * (k - 1) - 1) // s + 1, (W + 2 * p - d * (k - 1) - 1) // s + 1
    while Nb * Ho * Wo % B:
        Nb *= 2
    geom = hlq.hlq_conv_geom(Nb=Nb, H=H, W=W, C=C, O=B, kh=k, kw=k, stride_h=s, stride_w=s, pad_h=p, pad_w=p, dil_h=d, dil_w=d)
    _, _, N, I = hlq.hlq_conv_sizes(geom)
    print("image", c, dtype, B, "N", N, flush=True)
    X = torch.randn((Nb, H, W, C), generator=torch.Generator(device=DEV).manual_seed(7), device=DEV, dtype=torch.float32).to(dtype)
    cols = torch.empty((N, I), dtype=dtype, device=DEV)
    hlq.hlq_im2col(X, geom, cols)
    a, b = (torch.full((I, N // B * (B // 2)), 3.0, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    ca, cb = (torch.full((I, N // B * (B // 2)), 3.0, dtype=torch.float32, device=DEV) for _ in range(2))
    hlq.hlq_hla_project_basis(cols, B, B // 2, 0, a, ca)
    hlq.hlq_conv_compress_act(X, geom, B, B // 2, 0, b, cb)
    assert torch.equal(a, b) and torch.equal(ca, cb)
    assert float(cb.abs().max()) > 0
