"""Weight gradients that are stored and that are added to what is there, where tiles end inside the matrix and where rows of the result
are too long for offsets of 32 bits.  Reference: the product in fp64; the sums are in fp32, so the error of an element is some ulps of
the root sum of squares of its terms (one here, times the square root of the rows)."""
import pytest
import torch

import paper_2411_19460_amd as pk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("rows,K,N", [(256, 256, 256), (300, 264, 520), (64, 136, 8), (72, 520, 1032), (24, 2097168, 8)])
def test_weight_gradients(rows, K, N, accumulate):
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + N)
    x, d = (torch.randn((rows, n), generator=g, device="cuda").to(torch.bfloat16) for n in (K, N))
    w = torch.randn((N, K), generator=g, device="cuda").to(torch.bfloat16)
    start = torch.randn((N, K), generator=g, device="cuda")
    dw = start.clone()
    pk.ssd_linear_bwd(x, w, d, want_dx=False, flags=pk.SSD_FLAG_ACCUM_PARAM if accumulate else 0, dw=dw)
    torch.cuda.synchronize()
    want = d.double().T @ x.double() + (start.double() if accumulate else 0)
    assert float((dw.double() - want).abs().max()) <= 2 ** -20 * rows ** 0.5 * 8
