"""Launches that cover several checkpoint segments and ragged last chunks read and written in place:
every tensor against the oracle at the sizes where these can go wrong, with canaries behind the outputs."""
import numpy as np
import pytest
import torch

import paper_2411_19460_amd as pk
from oracle import ssd_ref
from parity_util import TOL, check, compare_all, dev_inputs, host, run_gpu, run_oracle
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


# 40 heads in segments of 1024 tokens: spans of four segments, so that ten segments run on two lanes (the caller's stream
# and one of the library's) with events between them.
LANES = dict(H=40, Q=256, seg=1024)


def _two_lanes(L, Bt=1, G=1, index=94):
    d = synth.make_layer_inputs(synth.SSDConfig("t", "bf16", Bt, L, LANES["H"], 64, 128, G, 1, L, index=index), with_states=True)
    return d, dev_inputs(d, "bf16")


def test_packed_sequences_on_two_lanes():
    """Packed sequences that start inside a chunk, on the boundaries of chunk, segment and span (4096 tokens), at the last token
    of a span and twice in a row."""
    L, Q, seg = 9 * 1024 + 5, LANES["Q"], LANES["seg"]
    d, dv = _two_lanes(L)
    reset = np.zeros((1, L), dtype=np.uint8)
    reset[0, [37, Q, Q + 1, seg, 4 * seg - 1, 4 * seg, 8 * seg + 700, L - 3]] = 1
    rdev = torch.from_numpy(reset).cuda()
    ins = [dv[k] for k in ("x", "dt", "A", "B", "C", "D")]
    y, fin, bnd = pk.ssd_fwd(*ins, Q, seg, dv["init_state"], seq_reset=rdev)
    g = pk.ssd_bwd(*ins, dv["dy"], Q, seg, dv["init_state"], dv["dfinal_state"], bnd, seq_reset=rdev)
    torch.cuda.synchronize()
    raw = [d[k] for k in ("x", "dt", "A", "B", "C", "D")]
    f = ssd_ref.ssd_fwd(*raw, d["init_state"], reset=reset)
    go = ssd_ref.ssd_bwd(*raw, d["dy"], d["init_state"], d["dfinal_state"], reset=reset)
    for k, got in (("y", y), ("final_state", fin)):
        check(k, host(got), f[k], TOL["bf16"])
    for k in ("dx", "ddt", "dA", "dB", "dC", "dD", "dinit_state"):
        check(k, host(g[k]), go[k], TOL["bf16"])


def test_checkpoints_and_chunk_states_on_two_lanes():
    """fp32 chunk states against the oracle; bf16 checkpoints round the same states and change nothing else of the forward
    pass, and the gradients by no more than that rounding allows."""
    L, Q, seg = 10 * 1024, LANES["Q"], LANES["seg"]
    d, _ = _two_lanes(L)
    dv, (y, fin, bnd, g) = compare_all(d, "bf16", Q, seg, flags=pk.SSD_FLAG_FP32_CHUNK_STATES)
    y32, fin32, bnd32, g32 = run_gpu(dv, Q, seg)
    y16, fin16, bnd16, g16 = run_gpu(dv, Q, seg, pk.SSD_FLAG_BF16_CHECKPOINTS)
    assert torch.equal(y16, y32) and torch.equal(fin16, fin32) and torch.equal(bnd16, bnd32.to(torch.bfloat16))
    for k in ("dx", "ddt", "dA", "dB", "dC", "dD", "dinit_state"):
        check(k, host(g16[k]), host(g32[k]), TOL["bf16"])


def test_two_lanes_replay_from_a_graph():
    """Forward and backward pass captured once, the library's streams and events with them; replays, with eager work in
    between, give the eager results bit for bit."""
    L, Q, seg, H = 9 * 1024 + 5, LANES["Q"], LANES["seg"], LANES["H"]
    _, dv = _two_lanes(L)
    shape = pk.make_shape(dv["x"], dv["B"], Q, seg)
    ws = [torch.empty(pk.ssd_workspace_bytes(shape, back), dtype=torch.uint8, device="cuda") for back in (False, True)]
    state = lambda *lead: torch.empty(lead + (H, 64, 128), device="cuda")  # noqa: E731
    out = {k: torch.empty_like(dv[v]) for k, v in (("y", "x"), ("dx", "x"), ("ddt", "dt"), ("dB", "B"), ("dC", "C"))}
    out.update(final_state=state(1), boundary_states=state(1, 10), dinit_state=state(1))
    dA, dD = torch.empty(H, device="cuda"), torch.empty(H, device="cuda")
    ins = [dv[k] for k in ("x", "dt", "A", "B", "C", "D")]

    def step():
        pk.ssd_fwd(*ins, Q, seg, dv["init_state"], 0, ws[0], out=out)
        pk.ssd_bwd(*ins, dv["dy"], Q, seg, dv["init_state"], dv["dfinal_state"], out["boundary_states"], 0, ws[1], dA, dD, out=out)

    step()
    torch.cuda.synchronize()
    got = {**out, "dA": dA, "dD": dD}
    want = {k: v.clone() for k, v in got.items()}
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.synchronize()
    for rep in range(3):
        for t in got.values():
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k, v in got.items():
            assert torch.equal(v, want[k]), (rep, k)


@pytest.mark.parametrize("case", [
    # dtype, L, H, P,   G, N,   Q,    segment: chunks of more than 256 tokens (several per thread), more than 64 channels, more
    # than 128 state columns
    ("f32", 2100, 2, 72, 1, 40, 1024, 1024),
    ("f32", 700, 4, 130, 2, 136, 320, 640),
    ("bf16", 1300, 3, 96, 1, 200, 520, 520),
])
def test_generic_kernels_beyond_their_usual_sizes(case):
    dtype, L, H, P, G, N, Q, seg = case
    d = synth.make_layer_inputs(synth.SSDConfig("t", dtype, 1, L, H, P, N, G, 1, L, index=95), with_states=True)
    dv = dev_inputs(d, dtype)
    y, fin, _, g = run_gpu(dv, Q, seg, pk.SSD_FLAG_GENERIC_KERNELS)
    f, go = run_oracle(d, None)
    for k, got, want in [("y", y, f["y"]), ("final_state", fin, f["final_state"])] + [
            (k, g[k], go[k]) for k in ("dx", "ddt", "dA", "dB", "dC", "dD", "dinit_state")]:
        check(k, host(got), want, TOL[dtype])


@pytest.mark.parametrize("L,H,seg,Q", [
    (16384, 80, 4096, 256),    # 5120 chunks of a head: the most that is one span
    (16385, 80, 8192, 256),    # one row more: lanes
    (39000, 32, 4992, 128),    # nearly as many in eight segments, ragged
    (40959, 32, 5120, 128),    # segments too long for eight of them to be one span: lanes
    (90000, 12, 22528, 256),   # few heads
    (122000, 9, 30720, 256),   # too few: lanes
])
def test_the_largest_single_span_against_one_segment(L, H, seg, Q):
    """Where the checkpoints fall does not change the result.  Tolerance: that of either run against the oracle."""
    g = torch.Generator(device="cuda").manual_seed(11)
    normal = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    x, Bm, Cm, dy = normal(1, L, H, 64), normal(1, L, 1, 128), normal(1, L, 1, 128), normal(1, L, H, 64)
    dt = (torch.rand((1, L, H), generator=g, device="cuda") * 0.1).to(torch.bfloat16)
    A, D = -torch.rand(H, generator=g, device="cuda") * 15 - 1, torch.randn(H, generator=g, device="cuda")
    out = []
    for s in (seg, -(-L // Q) * Q):
        y, fin, bnd = pk.ssd_fwd(x, dt, A, Bm, Cm, D, Q, s)
        b = pk.ssd_bwd(x, dt, A, Bm, Cm, D, dy, Q, s, boundary_states=bnd)
        out.append({"y": y, "final": fin, **{k: b[k] for k in ("dx", "ddt", "dA", "dB", "dC", "dD")}})
    torch.cuda.synchronize()
    for k, t in out[0].items():
        check(k, host(t), host(out[1][k]), TOL["bf16"])
