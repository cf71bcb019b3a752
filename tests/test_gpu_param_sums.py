"""dA and dD are summed by whichever chunk of a head ends last: more chunks than threads that sum them, one chunk, several
spans and lanes, workspaces full of anything."""
import pytest
import torch

import paper_2411_19460_amd as pk
from paper_2411_19460_amd import synth
from parity_util import TOL, check, dev_inputs, host, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # dtype, Bt, L,   H,  P,  N,   Q,  segment
    ("bf16", 1, 200, 3, 64, 128, 256, 256),        # one chunk
    ("bf16", 1, 3000, 24, 64, 128, 256, 4096),     # fewer chunks than a cache line has counts
    ("bf16", 2, 70 * 64 - 3, 5, 64, 128, 64, 8192),  # 140 chunks, summed by one wave; three waves too many in the launch
    ("bf16", 1, 9 * 1024 + 5, 40, 64, 128, 256, 1024),  # three spans on two lanes
    ("f32", 1, 2100, 2, 4, 4, 8, 4096),            # 263 chunks, summed by 256 threads
    ("f32", 1, 40, 3, 4, 4, 8, 8),                 # five spans' worth of segments
])
def test_the_last_chunk_sums(case):
    dtype, Bt, L, H, P, N, Q, seg = case
    d = synth.make_layer_inputs(synth.SSDConfig("t", dtype, Bt, L, H, P, N, 1, 1, L, index=97), with_states=True)
    dv = dev_inputs(d, dtype)
    ins = [dv[k] for k in ("x", "dt", "A", "B", "C", "D")]
    bnd = pk.ssd_fwd(*ins, Q, seg, dv["init_state"])[2]
    ws = torch.empty(pk.ssd_workspace_bytes(pk.make_shape(dv["x"], dv["B"], Q, seg), True), dtype=torch.uint8, device="cuda")
    runs = []
    for fill in (0, 1, 255):
        ws.fill_(fill)
        runs.append(pk.ssd_bwd(*ins, dv["dy"], Q, seg, dv["init_state"], dv["dfinal_state"], bnd, workspace=ws))
    torch.cuda.synchronize()
    first = {k: runs[0][k].clone() for k in ("dA", "dD")}
    for r in runs[1:]:
        assert all(torch.equal(r[k], first[k]) for k in first)
    again = {k: v.clone() for k, v in first.items()}  # on top of what is there: exactly twice as much
    pk.ssd_bwd(*ins, dv["dy"], Q, seg, dv["init_state"], dv["dfinal_state"], bnd, pk.SSD_FLAG_ACCUM_PARAM, ws, again["dA"], again["dD"])
    torch.cuda.synchronize()
    assert all(torch.equal(again[k], 2 * first[k]) for k in first)
    _, go = run_oracle(d, None)
    for k in first:
        check(k, host(first[k]), go[k], TOL[dtype])
    # dD = sum of dY . x: each of its L P products and sums rounds at most once to fp32, the order left open
    prod = dv["dy"].double() * dv["x"].double()
    bound = Bt * L * P * 2.0 ** -24 * prod.abs().sum((0, 1, 3))
    assert bool(((first["dD"].double() - prod.sum((0, 1, 3))).abs() <= bound).all())


@pytest.mark.parametrize("case", [
    ("bf16", 1, 600 * 64 + 7, 2, 64, 128, 64, 8192),   # 601 chunks: eight loads a lane in flight, and the rest
    ("bf16", 1, 512 * 64, 1, 64, 128, 64, 4096),       # exactly eight
    ("f32", 1, 2051 * 8 + 3, 1, 4, 4, 8, 4096),        # 2052 chunks, 256 threads
])
def test_more_chunks_than_loads_in_flight(case):
    test_the_last_chunk_sums(case)


def test_stack_with_less_than_a_line_of_state_per_head():
    """The counts of the heads lie in what one head's state of 2 x 3 elements leaves room for."""
    cfg = synth.SSDConfig("stack", "f32", 2, 96, 5, 2, 3, 1, 16, 32, nlayers=2, index=98)
    from test_gpu_stack import run_stack, stack_inputs
    from oracle import ssd_ref
    import numpy as np
    x0, dout, layers = stack_inputs(cfg)
    _, b = run_stack(cfg, x0, dout, layers, 1, 32)
    bo = ssd_ref.stack_bwd(ssd_ref.stack_fwd(x0, layers, segment=32)["xs"], layers, dout)
    for k in ("dA", "dD"):
        check(k, host(b[k]), np.stack([g[k] for g in bo["grads"]]), TOL["f32"])
