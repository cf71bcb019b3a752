"""Shape-generic kernels: chains of one to many contraction steps, last tiles of a chunk with up to 32 and with more rows (half a tile
has no second diagonal step), rows in and out of groups of four (16-byte loads or element by element), head slices that the two
slicings share and do not share; every tensor against the oracle."""
import pytest
import torch

import paper_2411_19460_amd as pk
from paper_2411_19460_amd import synth
from parity_util import check, dev_inputs, host, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

# The longest sums have Q + N terms; rounded one by one in fp32 they are off by at most that many half units in the last place.
HALF_ULP = 2.0 ** -24


@pytest.mark.parametrize("case", [
    # Bt, L, H, P, G, N, Q, segment
    (1, 1, 2, 4, 1, 4, 64, 64),           # one token
    (1, 32, 2, 16, 1, 16, 64, 64),        # half a tile exactly
    (1, 97, 2, 32, 1, 32, 128, 128),      # one row into the second half of the second tile
    (1, 160, 4, 64, 1, 96, 128, 128),     # the second chunk is half a tile; three state steps
    (1, 161, 3, 36, 1, 100, 96, 192),     # a tile and a half a chunk, one row past half a tile
    (2, 255, 24, 8, 1, 128, 256, 256),    # four slices of heads
    (1, 200, 6, 33, 2, 31, 100, 100),     # element by element, odd in every direction
])
def test_steps_and_halves_of_tiles(case):
    Bt, L, H, P, G, N, Q, seg = case
    d = synth.make_layer_inputs(synth.SSDConfig("t", "f32", Bt, L, H, P, N, G, 1, L, index=98), with_states=True)
    y, fin, _, g = run_gpu(dev_inputs(d, "f32"), Q, seg)
    f, go = run_oracle(d, None)
    tol = (Q + N) * HALF_ULP
    check("y", host(y), f["y"], tol)
    check("final_state", host(fin), f["final_state"], tol)
    for k in ("dx", "dB", "dC", "dinit_state"):
        check(k, host(g[k]), go[k], tol)
    for k in ("ddt", "dA", "dD"):         # sums over the chunk of such sums
        check(k, host(g[k]), go[k], 4 * tol)


def test_as_many_tiles_as_a_launch_has_threads_for():
    """2^24 workgroups of 256 threads in one span, more than one dimension of a grid takes: 1048576 tokens of 1024 heads.  A head's output
    does not depend on the others: the first and the last two against a call on them alone."""
    L, H, Q, g = 1 << 20, 1024, 128, torch.Generator(device="cuda")
    g.manual_seed(5)
    x = torch.randn((1, L, H, 1), generator=g, device="cuda", dtype=torch.bfloat16)
    dt = torch.rand((1, L, H), generator=g, device="cuda", dtype=torch.bfloat16) * 0.1 + 0.001
    A, D = -torch.rand(H, generator=g, device="cuda") * 8 - 1, torch.randn(H, generator=g, device="cuda")
    B, C = (torch.randn((1, L, 1, 1), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    y, fin, _ = pk.ssd_fwd(x, dt, A, B, C, D, Q)
    for h in (slice(0, 2), slice(H - 2, H)):
        y2, fin2, _ = pk.ssd_fwd(x[:, :, h].contiguous(), dt[:, :, h].contiguous(), A[h], B, C, D[h], Q)
        torch.cuda.synchronize()
        assert torch.equal(y[:, :, h], y2) and torch.equal(fin[:, h], fin2)
