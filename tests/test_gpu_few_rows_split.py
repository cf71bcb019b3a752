"""Products of few rows at the edges of how they are shared out: the vector ALUs (one and two rows) with one and two pieces of 512 k
a wave and with rows in turns, the matrix cores (from three rows on) with one and two pieces of 256 and in turns, columns of a
workgroup that are no whole tiles, a last workgroup with fewer of them, and more columns than one round of workgroups takes."""
import pytest
import torch

import paper_2411_19460_amd as pk
from oracle import linear_ref
from parity_util import TOL, check, host
from test_gpu_linear import dev, draw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 2, 3, 16])
@pytest.mark.parametrize("K,N", [
    (8, 8),
    (520, 136),       # a piece of eight k
    (2312, 4360),     # ten pieces of 256, 17 columns a workgroup or 18; the last has fewer
    (2568, 2568),     # two pieces of 256 a wave, the second one's most lanes without k
    (5128, 1032),     # two pieces of 512; pieces of 256 in turns
    (10248, 264),     # pieces of 512 in turns
    (264, 49160),     # more columns than one round
    (2560, 16392),    # the same with ten waves a workgroup
])
def test_few_rows(rows, K, N):
    """Tolerance of a bf16 product: sums in fp32, one rounding of the result (half an ulp, 2^-9 of it)."""
    x, w, _ = draw(7, rows, K, N)
    out = pk.ssd_linear_fwd(dev(x), dev(w))
    torch.cuda.synchronize()
    check("out", host(out), linear_ref.linear_fwd(x, w), TOL["bf16"])
