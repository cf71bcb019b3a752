"""What a stack of blocks takes in scratch: the activations of one grid cell, whatever the length of the sequence (host only: the
library's own size queries)."""
import ctypes

import pytest

import paper_2411_19460_amd as pk
from paper_2411_19460_amd import binding

P, N = 64, 128


def _stack(H, L, seg, nl=2, l=1, Q=256, G=1, hd=P, n=N, dm=None):
    return binding.magc_blockstack_shape_t(binding.magc_block_shape_t(dm or 32 * H, H, hd, G, n, Q, 1e-5, L, seg), nl, l)


def need(*a, back=False, **k):
    return int(pk.lib().magc_blockstack_workspace_bytes(ctypes.byref(_stack(*a, **k)), int(back)))


def block_need(sh, back):
    one = binding.magc_block_shape_t.from_buffer_copy(sh.block)
    one.seqlen = one.segment
    return int(pk.lib().magc_block_workspace_bytes(ctypes.byref(one), int(back)))


def sizes(H, Q=256, G=1, hd=P, n=N, dm=None):
    """Bytes: of a kept layer input and of what a cell keeps, per layer and token; of both states of a layer; of their adjoints."""
    dm, di, gn = dm or 32 * H, H * hd, G * n
    conv, d_in = di + 2 * gn, 2 * di + 2 * gn + H
    return dm * 2, (dm + d_in + di) * 2, H * hd * n * 4 + 3 * conv * 2, H * hd * n * 4 + 3 * conv * 4


@pytest.mark.parametrize("case", [
    # heads, tokens, segment, layers, interval, further dimensions
    (24, 262144, 1024, 24, 24, {}),
    (80, 65536, 256, 8, 8, {}),
    (80, 16384, 4096, 2, 1, {}),
    (24, 65536, 4096, 8, 4, {}),
    (8, 400000, 2, 1, 1, dict(Q=2, n=256)),            # short chunks, large states
    (8, 5000000, 4096, 1, 1, dict(hd=1, G=8, n=1, dm=8)),  # the narrowest block there is
])
def test_scratch_is_that_of_one_cell(case):
    H, L, seg, nl, l, more = case
    c_l, c_grid, c_s, c_adj = sizes(H, **more)
    sh = _stack(H, L, seg, nl, l, **more)
    # a cell's kept tensors, the block's own scratch, four buffers of activations, the adjoints of all layers, sixteen convolution
    # states of a generation step; every array on a boundary of 256 bytes
    fixed = 4 * seg * c_l + 17 * c_s + 256 * (4 * nl + 16)
    assert 0 < need(H, L, seg, nl, l, **more) <= block_need(sh, False) + fixed
    assert 0 < need(H, L, seg, nl, l, back=True, **more) <= l * seg * c_grid + max(block_need(sh, b) for b in (False, True)) + 2 * nl * c_adj + fixed
    for back in (False, True):       # and nothing else: not the length of the sequence
        assert len({need(H, k * seg, seg, nl, l, back=back, **more) for k in (16, 17, 64, 1000)}) == 1


@pytest.mark.parametrize("H", [24, 80])
@pytest.mark.parametrize("nl", [24, 64])
def test_what_the_planner_chooses_fits_what_it_says(H, nl):
    """Checkpoints and scratch of the grids that magc_plan returns, for the least memory and for budgets above it, against its
    own total.  The model has no term for the state adjoints of the layers, nor for the buffers that do not grow with the
    interval, and its scratch term is linear in the segment: what a block really takes at that segment is added."""
    c_l, c_grid, c_s, c_adj = sizes(H)
    c_state = block_need(_stack(H, 4096, 4096), True) // 4096
    for S in (4096, 16384, 65536, 262144):
        plan = lambda budget: pk.magc_plan(nl, S, c_l, c_s, c_grid, c_state, s_multiple=256, budget=budget, integer_counts=True)  # noqa: E731
        least = plan(0.0)[1]["m_total"]
        for times in (0.0, 1.5, 3.0):
            rc, p = plan(times * least)
            assert rc == 0
            l, s = p["l"], p["s"]
            kept = nl * -(-S // s) * c_s + (-(-nl // l) - 1) * S * c_l
            scratch = max(need(H, S, s, nl, l, back=b) for b in (False, True))
            short = max(0, max(block_need(_stack(H, n, n), True) for n in {s, S % s or s}) - s * c_state)
            assert kept + scratch <= p["m_total"] + short + 2 * nl * c_adj + 4 * s * c_l + 17 * c_s + 65536, (S, times, l, s)


@pytest.mark.parametrize("dims", [dict(Q=64), dict(Q=128), dict(Q=256), dict(Q=128, G=2), dict(Q=256, hd=16, n=16)])
def test_scratch_for_the_longest_sequence_serves_shorter_ones(dims):
    Q = dims["Q"]
    for H in (8, 24, 32, 80):
        for nseg in (1, 2, 4):
            for back in (False, True):
                got = [need(H, L, nseg * Q, back=back, **dims) for L in range(Q // 2, 48 * Q, Q // 2)]
                assert min(got) > 0 and got == sorted(got), (H, nseg, back)


def uses(limit, *a, keep, **k):
    """What a forward pass uses of a workspace of `limit` bytes."""
    return int(pk.lib().magc_blockstack_pass_bytes(ctypes.byref(_stack(*a, **k)), int(keep), limit))


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("dims", [dict(), dict(Q=128, G=2), dict(Q=64), dict(hd=16, n=16), dict(Q=2, hd=16, n=256), dict(Q=1, hd=1, G=8, n=1, dm=8),
                                  dict(dm=8192, hd=8, n=8)])
def test_a_forward_pass_keeps_to_the_workspace_that_it_is_given(dims, keep):
    """The least that the queries ask for is enough at every length, what is used never exceeds what is given, and more is used
    only up to what a pass of 8192 (nothing kept: 16384) rows of the 2.7B width has use for."""
    Q, most = dims.get("Q", 256), {}
    for H in (8, 24, 80):
        dm, di, gn = dims.get("dm", 32 * H), H * dims.get("hd", P), dims.get("G", 1) * dims.get("n", N)
        for seg in (Q, 3 * Q, 16 * Q):
            for L in (1, seg, seg + 1, 2 * seg - 1, 5 * seg + 17, 40 * seg + 3):
                least, got = need(H, L, seg, **dims), []
                for times in (0.0, 0.5, 1.0, 1.3, 2.0, 3.7, 1000.0):
                    limit = int(times * least)
                    got.append(uses(limit, H, L, seg, keep=keep, **dims))
                    assert 0 < got[-1] <= max(limit, least), (H, seg, L, times)
                assert got[0] == got[1] == got[2]
                if L <= seg:
                    assert set(got) == {least}       # one segment: nothing to join
                elif seg >= 16:                      # the tokens of a pass, by the projection's output alone
                    rows = (8192 if keep else 16384) * 10576 // max(2 * di + 2 * gn + H, dm)
                    assert got[-1] <= 2 * least * max(1, -(-min(L, rows) // seg)), (H, seg, L)


def test_a_prompt_of_any_length_runs_in_pieces_that_every_step_takes():
    """The narrowest block there is: the convolution takes 65535 x 64 tokens a call."""
    sh = dict(Q=1, hd=1, G=8, n=1, dm=8)
    some, many = (uses(1 << 60, 8, n, 4096, keep=False, nl=1, **sh) for n in (65535 * 64, 5000000))
    assert 0 < many <= some
