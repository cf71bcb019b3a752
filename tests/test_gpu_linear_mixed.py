"""The forward product where it takes tiles of two widths: each pair of widths, rows and columns that end inside a tile, a contraction that
is no multiple of a K step, operands and result as column slices of wider tensors.  The result is that of fp32 sums rounded once, whatever
the tile, so a reference product in fp32 decides; its own sums differ by a few ulps of fp32."""
import pytest
import torch

import paper_2411_19460_amd as pk
from parity_util import TOL, check, host
from test_gpu_linear import in_wider

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,K,N,wide", [
    (4096, 264, 10576, False),   # 256 and 192 columns a tile: two rounds of the one and one of the other
    (4000, 200, 10568, True),
    (8192, 320, 2560, False),    # 192 and 128
    (4100, 136, 4384, True),
    (16384, 64, 2560, False),    # 256 and 192: one round and two
    (16300, 72, 10304, True),    # eight and three
])
def test_two_widths(rows, K, N, wide):
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    x = torch.randn((rows, K), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((N, K), generator=g, device="cuda") * K ** -0.5).to(torch.bfloat16)
    out = pk.ssd_linear_fwd(in_wider(x, K + 48, 16) if wide else x, w)
    torch.cuda.synchronize()
    want = x.float() @ w.float().T
    worst = ((out.float() - want).abs() / (want.abs() + 1)).max()
    assert worst <= 2 ** -8, worst          # a rounding of the result is half of this
    check("out", host(out[-300:]), host(want[-300:]), TOL["bf16"])


@pytest.mark.parametrize("rows,K,N", [(4000, 200, 10568), (4100, 136, 4384), (8192, 72, 2560), (16300, 72, 10304)])
def test_result_inside_a_wider_tensor(rows, K, N):
    """The second width's origin and both widths' right edges in rows that go on behind them: the columns around the result, and a row
    in front of it and one behind, stay as they are, and the result is that of a dense one, bit by bit."""
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    x = torch.randn((rows, K), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((N, K), generator=g, device="cuda") * K ** -0.5).to(torch.bfloat16)
    wide = torch.full((rows + 2, N + 40), 7.0, device="cuda", dtype=torch.bfloat16)
    out = wide[1:-1, 16:16 + N]
    pk.ssd_linear_fwd(x, w, out=out)
    dense = pk.ssd_linear_fwd(x, w)
    torch.cuda.synchronize()
    assert torch.equal(out, dense)
    around = wide.clone()
    around[1:-1, 16:16 + N] = 7.0
    assert bool((around == 7.0).all())
