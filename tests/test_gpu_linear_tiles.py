"""The projections at the sizes where their tile width changes (128, 192, 256 columns) and at the edges of these tiles: K
steps that are too few for the straight-line loop, exactly as many, and with a remainder; last tiles of a few rows or
columns, read through bounded descriptors; views with wider rows.  Against the fp64 oracle."""
import pytest
import torch

import paper_2411_19460_amd as pk
from test_gpu_linear import test_linear_forward_backward as check_linear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # rows, in_dim, out_dim, operands as column slices of wider tensors
    (130, 184, 40008, False),      # 192 columns forward; K of two whole steps and a remainder
    (270, 200, 20008, True),       # 192 columns forward; three steps and a remainder, views
    (450, 192, 25000, True),       # 256 columns forward; exactly three steps
    (257, 1024, 136, True),        # 128 columns; one row and eight columns beyond a tile
    (2049, 328, 264, False),       # dw over many rows with a remainder of one
])
def test_linear_tile_widths(case):
    check_linear(case)


@pytest.mark.parametrize("case", [
    # K steps of 64 around the straight-line loop's four, in each product's contraction, at each width
    (256, 256, 256, False),        # exactly four steps everywhere
    (264, 320, 40008, True),       # five; 192 columns forward
    (328, 248, 25000, False),      # three and a remainder forward, five and a remainder for dw
    (8200, 312, 600, False),       # four and a remainder; dw over 128 steps and a remainder of eight
    (257, 1016, 520, True),        # an odd number of rows as dw's contraction
])
def test_linear_loop_edges(case):
    check_linear(case)


@pytest.mark.parametrize("shape", [(20, 328, 264), (40, 64, 136)])
def test_linear_rows_beyond_32_bit_offsets(shape):
    """Row strides past the reach of 32-bit offsets inside a tile (the operands then pass through registers): same bits as
    dense rows."""
    rows, K, N = shape
    g = torch.Generator(device="cuda").manual_seed(5)
    draw = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    x, w, dout = draw(rows, K), draw(N, K), draw(rows, N)
    far = []
    for t in (x, dout):
        wide = torch.empty((rows, (1 << 22) + 8), dtype=torch.bfloat16, device="cuda")
        far.append(wide[:, 8:8 + t.shape[1]])
        far[-1].copy_(t)
    want, got = pk.ssd_linear_bwd(x, w, dout), pk.ssd_linear_bwd(far[0], w, far[1])
    assert torch.equal(pk.ssd_linear_fwd(x, w), pk.ssd_linear_fwd(far[0], w))
    assert torch.equal(want["dx"], got["dx"]) and torch.equal(want["dw"], got["dw"])


def test_linear_weight_gradient_is_added_to():
    """dw accumulated over two calls, tiles cut at both edges: the sum of the two products."""
    g = torch.Generator(device="cuda").manual_seed(6)
    x, dout = (torch.randn((300, n), generator=g, device="cuda").to(torch.bfloat16) for n in (392, 776))
    w = torch.zeros((776, 392), dtype=torch.bfloat16, device="cuda")
    one = pk.ssd_linear_bwd(x, w, dout, want_dx=False)["dw"]
    acc = one.clone()
    pk.ssd_linear_bwd(x, w, dout, want_dx=False, dw=acc, flags=pk.SSD_FLAG_ACCUM_PARAM)
    assert torch.equal(acc, one + one)


@pytest.mark.parametrize("shape", [
    # rows, in_dim, out_dim: each pair of tile widths (input's, weights' gradient), each product first, tiles cut at the edges
    (72, 264, 136),       # 256, 128; the weights' first
    (1300, 2568, 2056),   # 256, 128; the input's first
    (72, 264, 520),       # 128, 128; the weights'
    (72, 264, 1032),      # 128, 128; the input's
    (72, 264, 2056),      # 128, 256; the input's
    (1000, 2568, 2056),   # 128, 256; the weights'
    (2049, 1544, 3080),   # 256, 256; the input's
    (2049, 2568, 2056),   # 256, 256; the weights'
])
def test_linear_gradients_of_one_launch(shape):
    """Both gradients of a call against each of them alone: same bits, as a result is summed in the same order at any width."""
    rows, K, N = shape
    g = torch.Generator(device="cuda").manual_seed(7)
    x, w, dout = (torch.randn(s, generator=g, device="cuda").to(torch.bfloat16) for s in ((rows, K), (N, K), (rows, N)))
    both = pk.ssd_linear_bwd(x, w, dout)
    assert torch.equal(both["dx"], pk.ssd_linear_bwd(x, w, dout, want_dw=False)["dx"])
    assert torch.equal(both["dw"], pk.ssd_linear_bwd(x, w, dout, want_dx=False)["dw"])
