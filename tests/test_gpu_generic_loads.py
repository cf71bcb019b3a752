"""Shape-generic kernels: how operands leave memory.  Sizes, strides and addresses in fours, in words and in neither, rows whose last
elements are one to three behind a group of four, the shortest rows that are asked for in fours and shorter ones."""
import pytest
import torch

import paper_2411_19460_amd as pk
from paper_2411_19460_amd import synth
from parity_util import TOL, check, dev_inputs, host, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

# The longest sums have Q + N terms; rounded one by one in fp32 they are off by at most that many half units in the last place.
HALF_ULP = 2.0 ** -24
GENERIC = pk.SSD_FLAG_GENERIC_KERNELS


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [
    # Bt, L, H, P, G, N, Q, segment
    (1, 150, 2, 64, 1, 128, 63, 126),     # only the chunk length is odd
    (1, 203, 4, 32, 2, 64, 101, 101),
    (1, 203, 4, 64, 1, 128, 130, 130),    # two elements behind a group of four, and behind whole tiles
    (1, 140, 2, 36, 1, 30, 70, 70),       # even
    (2, 97, 3, 33, 1, 35, 67, 67),        # one, three, three behind
    (1, 131, 2, 67, 1, 65, 131, 131),     # a second tile of three columns, of one, a third of three
    (1, 19, 2, 4, 1, 5, 6, 12),           # the shortest rows
    (1, 19, 2, 5, 1, 4, 7, 7),
    (1, 41, 2, 3, 1, 128, 64, 64),        # shorter ones
    (1, 41, 2, 64, 1, 2, 33, 33),
    (1, 10, 1, 16, 1, 16, 3, 6),
])
def test_rows_of_any_length(case, dtype):
    Bt, L, H, P, G, N, Q, seg = case
    d = synth.make_layer_inputs(synth.SSDConfig("t", dtype, Bt, L, H, P, N, G, 1, L, index=99), with_states=True)
    y, fin, _, g = run_gpu(dev_inputs(d, dtype), Q, seg, GENERIC if dtype == "bf16" else 0)
    f, go = run_oracle(d, None)
    tol = (Q + N) * HALF_ULP if dtype == "f32" else TOL["bf16"]
    check("y", host(y), f["y"], tol)
    check("final_state", host(fin), f["final_state"], tol)
    for k in ("dx", "dB", "dC", "dinit_state"):
        check(k, host(g[k]), go[k], tol)
    for k in ("ddt", "dA", "dD"):         # sums over the chunk of such sums
        check(k, host(g[k]), go[k], 4 * tol if dtype == "f32" else tol)


@pytest.mark.parametrize("dtype,off", [(torch.float32, 1), (torch.float32, 2), (torch.bfloat16, 1), (torch.bfloat16, 2)])
@pytest.mark.parametrize("which", [(0, 3, 4, 6), (0,), (3,), (6,)])
def test_the_address_does_not_matter(dtype, off, which):
    """x, B, C and dY that begin off a group of four elements: the same sums in the same order, bit by bit."""
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    normal = lambda *s: torch.randn(s, generator=g, device="cuda").to(dtype)  # noqa: E731
    Bt, L, H, P, G, N, Q = 2, 300, 6, 36, 2, 68, 128
    args = [normal(Bt, L, H, P), (torch.rand((Bt, L, H), generator=g, device="cuda") * 0.1).to(dtype), -torch.rand(H, generator=g, device="cuda") * 8 - 1,
            normal(Bt, L, G, N) / 8, normal(Bt, L, G, N) / 8, torch.randn(H, generator=g, device="cuda"), normal(Bt, L, H, P)]

    def run(a):
        y, fin, bnd = pk.ssd_fwd(*a[:6], Q, None, flags=GENERIC)
        return [y, fin, *pk.ssd_bwd(*a, Q, None, boundary_states=bnd, flags=GENERIC).values()]

    want = run(args)
    for i in which:
        wide = torch.empty(args[i].numel() + off, device="cuda", dtype=dtype)
        wide[off:] = args[i].reshape(-1)
        args[i] = wide[off:].view(args[i].shape)
        assert args[i].data_ptr() % (4 * args[i].element_size())
    got = run(args)
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)
