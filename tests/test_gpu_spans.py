"""Launches that cover several checkpoint segments and ragged last chunks read and written in place:
every tensor against the oracle at the sizes where these can go wrong, with canaries behind the outputs."""
import pytest
import torch

import paper_2411_19460_amd as pk
from oracle import ssd_ref
from parity_util import TOL, check, dev_inputs, host, run_oracle
from paper_2411_19460_amd import synth

pytestmark = pytest.mark.gpu


def _guarded(like, pad=4096):
    """A tensor of `like`'s shape inside a larger buffer of NaNs, and the part behind it."""
    buf = torch.full((like.numel() + pad,), float("nan"), dtype=like.dtype, device="cuda")
    return buf[:like.numel()].view(like.shape), buf[like.numel():]


@pytest.mark.parametrize("case", [
    # dtype, Bt, L,    H,  P,  G, N,   Q,   segment
    ("bf16", 1, 1, 2, 64, 1, 128, 256, 256),            # one token
    ("bf16", 2, 255, 2, 64, 2, 128, 256, 256),          # one row short of a chunk
    ("bf16", 1, 257, 2, 64, 1, 128, 256, 256),          # a chunk of one row, in a segment of its own
    ("bf16", 1, 19 * 256 + 33, 4, 64, 1, 128, 256, 256),   # three spans of up to eight segments, one lane
    ("bf16", 1, 9 * 1024 + 5, 40, 64, 1, 128, 256, 1024),  # three spans of four segments on two lanes
    ("bf16", 2, 3077, 4, 64, 2, 128, 128, 1024),        # chunks of 128, one span of four segments
    ("bf16", 1, 130, 3, 64, 1, 128, 64, 128),           # chunk 64
    ("f32", 1, 11 * 64 + 7, 3, 16, 1, 24, 64, 64),      # shape-generic kernels, two spans
])
def test_spans_and_ragged_tails(case):
    dtype, Bt, L, H, P, G, N, Q, seg = case
    cfg = synth.SSDConfig("t", dtype, Bt, L, H, P, N, G, 1, L, index=90)
    d = synth.make_layer_inputs(cfg, with_states=True)
    dv = dev_inputs(d, dtype)
    ins = [dv[k] for k in ("x", "dt", "A", "B", "C", "D")]
    nseg = -(-L // seg)
    shapes = {"y": dv["x"], "final_state": dv["init_state"], "boundary_states": torch.empty((Bt, nseg, H, P, N), device="cuda"),
              "dx": dv["x"], "ddt": dv["dt"], "dB": dv["B"], "dC": dv["C"], "dinit_state": dv["init_state"]}
    out = {k: _guarded(t) for k, t in shapes.items()}
    o = {k: t for k, (t, _) in out.items()}
    _, _, bnd = pk.ssd_fwd(*ins, Q, seg, dv["init_state"], out=o)
    g = pk.ssd_bwd(*ins, dv["dy"], Q, seg, dv["init_state"], dv["dfinal_state"], bnd, out=o)
    torch.cuda.synchronize()
    f, go = run_oracle(d, None)
    for k in ("y", "final_state"):
        check(k, host(o[k]), f[k], TOL[dtype])
    for k in {0, 1, nseg // 2, nseg - 1} & set(range(nseg)):   # the state entering segment k
        n = k * seg
        want = ssd_ref.ssd_fwd(*[d[v][:, :n] if v not in ("A", "D") else d[v] for v in ("x", "dt", "A", "B", "C", "D")], d["init_state"])
        check(f"boundary_states[{k}]", host(o["boundary_states"][:, k]), want["final_state"] if n else d["init_state"], TOL[dtype])
    for k in ("dx", "ddt", "dA", "dB", "dC", "dD", "dinit_state"):
        check(k, host(g[k]), go[k], TOL[dtype])
    for k, (_, guard) in out.items():
        assert bool(torch.isnan(guard).all()), f"{k}: written beyond its end"
