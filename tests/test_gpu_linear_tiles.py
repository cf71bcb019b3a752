"""The projections at the sizes where their tile width changes (128, 192, 256 columns) and at the edges of these tiles: K
steps that are too few for the straight-line loop, exactly as many, and with a remainder; last tiles of a few rows or
columns, read through bounded descriptors; views with wider rows.  Against the fp64 oracle."""
import pytest

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
