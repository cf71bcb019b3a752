"""The convolution at the edges of its runs of tokens: sequences shorter than a run, one token on either side of one and of several, a last
run that starts inside the one before it, the longest runs, workgroups whose last waves have no tokens, channels that leave lanes idle.
Against the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_2411_19460_amd as pk
from oracle import conv_ref
from parity_util import TOL, check, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,Bt,C,lengths", [
    ("bf16", 1, 264, (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 16, 17, 20, 21, 23)),   # runs of eight and five tokens
    ("f32", 2, 36, (1, 4, 5, 6, 8, 9, 21, 22)),
    ("bf16", 1, 5, (4, 5, 6, 7, 8, 9, 25)),                                          # a channel a thread
    ("bf16", 160, 256, (1793, 1801, 2100)),                                          # runs of 64 and 69
    ("bf16", 40, 512, (1001,)),                                                      # runs in between
])
@pytest.mark.parametrize("states", [True, False])
def test_runs(dtype, Bt, C, lengths, states):
    """Only the first and the last sequence have a gradient, so that the oracle needs these two alone.  Tolerance as for every use of the
    convolution."""
    T = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(C)
    normal = lambda *shape, t=torch.float32: torch.randn(shape, generator=g, device="cuda", dtype=t)  # noqa: E731
    w, bias = normal(C, 4) * 0.5, normal(C)
    some = sorted({0, Bt - 1})
    pick = lambda t: host(t[some])  # noqa: E731
    for L in lengths:
        u, dout = normal(Bt, L, C, t=T), normal(Bt, L, C, t=T)
        st, dso = (normal(Bt, 3, C, t=T), normal(Bt, 3, C)) if states else (None, None)
        dout[1:Bt - 1] = 0
        if states:
            dso[1:Bt - 1] = 0
        out, so = pk.ssd_conv1d_fwd(u, w, bias, st)
        got = pk.ssd_conv1d_bwd(u, w, bias, st, dout, dso)
        torch.cuda.synchronize()
        st_h = pick(st) if states else np.zeros((len(some), 3, C))
        dso_h = pick(dso) if states else np.zeros((len(some), 3, C))
        f = conv_ref.conv1d_silu_fwd(pick(u), host(w), host(bias), st_h)
        go = conv_ref.conv1d_silu_bwd(pick(u), host(w), host(bias), st_h, pick(dout), dso_h)
        check(f"{L} out", pick(out), f["out"], TOL[dtype])
        assert np.array_equal(pick(so), f["state_out"]), L
        check(f"{L} du", pick(got["du"]), go["du"], TOL[dtype])
        check(f"{L} dstate_in", pick(got["dstate_in"]), go["dstate_in"], TOL[dtype])
        check(f"{L} dw", host(got["dw"]), go["dw"], TOL[dtype])
        check(f"{L} dbias", host(got["dbias"]), go["dbias"], TOL[dtype])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("C", [1, 2, 3, 4])
def test_few_channels(dtype, C):
    """Fewer channels than a thread's share of a wider tensor."""
    test_runs(dtype, 2, C, (1, 2, 7, 8, 9, 40, 300), True)


@pytest.mark.parametrize("dtype,Bt,C,L", [("bf16", 7, 264, 1), ("bf16", 9, 2048, 64), ("f32", 6, 1536, 30), ("bf16", 5, 8, 0), ("bf16", 258, 512, 100)])
def test_waves_of_a_workgroup_on_several_sequences(dtype, Bt, C, L):
    """A sequence with fewer runs than a workgroup has waves shares it with its neighbours: every sequence has gradients, the last workgroup
    waves without any.  Tolerance as for every use of the convolution."""
    T = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(L)
    normal = lambda *shape, t=torch.float32: torch.randn(shape, generator=g, device="cuda", dtype=t)  # noqa: E731
    w, bias, u, dout, st, dso = normal(C, 4) * 0.5, normal(C), normal(Bt, L, C, t=T), normal(Bt, L, C, t=T), normal(Bt, 3, C, t=T), normal(Bt, 3, C)
    got = pk.ssd_conv1d_bwd(u, w, bias, st, dout, dso)
    torch.cuda.synchronize()
    go = conv_ref.conv1d_silu_bwd(host(u), host(w), host(bias), host(st), host(dout), host(dso))
    for k in ("du", "dstate_in", "dw", "dbias"):
        if got[k].numel():
            check(k, host(got[k]), go[k], TOL[dtype])


@pytest.mark.parametrize("dtype,Bt,C", [("f32", 1400, 512), ("bf16", 700, 2048), ("bf16", 520, 645)])
def test_sequences_of_part_of_a_run(dtype, Bt, C):
    """So many sequences that one run is a sequence, which ends inside a group of four or eight rows, or at its end."""
    test_runs(dtype, Bt, C, (1, 3, 4, 5, 9, 12, 13, 20, 21, 45, 63), True)
