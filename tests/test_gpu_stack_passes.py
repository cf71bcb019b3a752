"""The forward passes of a stack of blocks take as many tokens at a time as the workspace they are given has room for: output,
checkpoints and states are the same bits whatever that is.  (The last piece of every sequence here has more tokens than the kernels
of a few rows take, which round elsewhere.)"""
import ctypes

import pytest
import torch

import paper_2411_19460_amd as pk
from paper_2411_19460_amd import binding
from test_gpu_rows_together import _input, _layers

pytestmark = pytest.mark.gpu

CASES = [
    # d_model, H, P, G, N, chunk, segment, L, layers, interval
    (128, 8, 64, 1, 128, 128, 256, 2900, 3, 2),
    (128, 8, 64, 2, 128, 256, 512, 4096, 2, 2),       # whole segments
    (768, 24, 64, 1, 128, 256, 1024, 5001, 2, 1),
    (64, 8, 16, 1, 16, 64, 128, 1000, 3, 3),
    (512, 8, 16, 1, 16, 64, 128, 1000, 2, 1),         # a model wider than its heads: the block's output is longer than y
]


def _stack_layers(NL, *dims):
    """Two layers without the pre-norm, three with it."""
    return [{k: v for k, v in p.items() if k != "pre_norm_w" or NL == 3} for p in _layers(NL, *dims)]


def _sizes(x0, NL, H, P, G, N, Q, seg, keep):
    """Scratch for one of the caller's segments, and up to what a pass has use for."""
    sh = binding.magc_blockstack_shape_t(binding.magc_block_shape_t(x0.shape[1], H, P, G, N, Q, 1e-5, x0.shape[0], seg), NL, 1)
    least = int(pk.lib().magc_blockstack_workspace_bytes(ctypes.byref(sh), 0))
    most = int(pk.lib().magc_blockstack_pass_bytes(ctypes.byref(sh), int(keep), 1 << 60))
    sizes = [least, least * 5 // 4, least * 2, max(least, most), 4 * most + 4096]
    used = {int(pk.lib().magc_blockstack_pass_bytes(ctypes.byref(sh), int(keep), n)) for n in sizes}
    assert len(used) >= 3, used
    return sizes


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("shift", [0, 4])      # of the output from a boundary of 16 bytes, in elements
def test_inference_in_any_workspace(case, shift):
    dm, H, P, G, N, Q, seg, L, NL, _ = case
    layers, x0 = _stack_layers(NL, dm, H, P, G, N), _input(L, dm, 4)
    want = None
    for n in _sizes(x0, NL, H, P, G, N, Q, seg, False):
        ws = torch.full((n,), 255, dtype=torch.uint8, device="cuda")      # NaN wherever something unwritten is read
        out = torch.empty(L * dm + 8, dtype=torch.bfloat16, device="cuda")[shift:shift + L * dm].view(L, dm)
        st = pk.magc_blockstack_infer(x0, layers, H, P, G, N, Q, seg, out=out, workspace=ws)
        assert st["workspace"] is ws
        got = [st[k].clone() for k in ("out", "ssm_state", "conv_state")]
        want = want or got
        assert all(torch.equal(a, b) for a, b in zip(got, want)), n
    if shift == 0:
        xio = x0.clone()                                                  # output over the input
        st = pk.magc_blockstack_infer(xio, layers, H, P, G, N, Q, seg, out=xio)
        assert all(torch.equal(st[k], b) for k, b in zip(("out", "ssm_state", "conv_state"), want))


@pytest.mark.parametrize("case", CASES)
def test_checkpoints_in_any_workspace(case):
    dm, H, P, G, N, Q, seg, L, NL, l = case
    layers, x0 = _stack_layers(NL, dm, H, P, G, N), _input(L, dm, 5)
    sh, pars, _, nseg, conv_dim = binding._blockstack_setup(x0, layers, H, P, G, N, Q, seg, l, 1e-5)
    want = None
    for n in _sizes(x0, NL, H, P, G, N, Q, seg, True):
        ws = torch.full((n,), 255, dtype=torch.uint8, device="cuda")
        out, l_ckpt = torch.empty_like(x0), torch.zeros((-(-NL // l), L, dm), dtype=torch.bfloat16, device="cuda")
        ssm = torch.zeros((NL, nseg, H, P, N), device="cuda")
        conv = torch.zeros((NL, nseg, 3, conv_dim), dtype=torch.bfloat16, device="cuda")
        rc = pk.lib().magc_blockstack_fwd(ctypes.byref(sh), pars, x0.data_ptr(), out.data_ptr(), l_ckpt.data_ptr(), ssm.data_ptr(), conv.data_ptr(),
                                          ws.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        got = (out, l_ckpt, ssm, conv)
        want = want or got
        assert all(torch.equal(a, b) for a, b in zip(got, want)), n
    st = pk.magc_blockstack_infer(x0, layers, H, P, G, N, Q, seg)
    assert torch.equal(st["out"], want[0])


def test_pieces_that_end_in_a_few_tokens():
    """A last piece of a few tokens takes the kernels of a few rows, in a workspace laid out for many."""
    dm, H, P, G, N, Q, seg, NL = 128, 8, 64, 1, 128, 128, 256, 2
    layers = _layers(NL, dm, H, P, G, N)
    for L in (257, 256 + 16, 3 * 256 + 5, 5 * 128 + 1):
        x0 = _input(L, dm, 6)
        whole = pk.magc_blockstack_infer(x0, layers, H, P, G, N, Q, -(-L // Q) * Q)
        st = pk.magc_blockstack_infer(x0, layers, H, P, G, N, Q, seg)
        for k, band in (("out", 2.0 ** -6), ("ssm_state", 2.0 ** -7), ("conv_state", 2.0 ** -7)):   # the bands of the grid's own tests
            a, b = st[k].float(), whole[k].float()
            assert float((a - b).abs().max()) <= band * float(b.abs().max()), (L, k)
