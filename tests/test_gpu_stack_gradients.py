"""The backward pass of a stack of blocks walks the caller's segments: its parameter gradients are those of the single block, bit
for bit, and the partial sums of its score gradients are stored as those of a scan of one segment."""
import numpy as np
import pytest
import torch

import paper_2411_19460_amd as pk
from oracle import block_ref, norm_ref, ssd_ref
from paper_2411_19460_amd import synth
from parity_util import host
from test_gpu_block import BF, GRADS, dev_bf16, draw, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # d_model, H, P, G, N, chunk, segment, L
    (768, 24, 64, 1, 128, 256, 4096, 12288),
    (1024, 32, 64, 2, 128, 256, 1024, 5001),
    (128, 8, 64, 1, 128, 128, 256, 1200),
    (64, 8, 16, 1, 16, 64, 128, 700),
])
def test_a_stack_of_one_block_has_the_gradients_of_the_block(case):
    dm, H, P, G, N, Q, seg, L = case
    d = draw(91, L, dm, H, P, G, N)
    u, dout, par = dev_bf16(d["u"]), dev_bf16(d["dout"]), to_dev(d["p"])
    f = pk.magc_block_fwd(u, par, H, P, G, N, Q, seg)
    g = pk.magc_block_bwd(u, par, dout, f["ssm_ckpt"], f["conv_ckpt"], H, P, G, N, Q, seg)
    fs = pk.magc_blockstack_fwd(u, [par], H, P, G, N, Q, seg, 1)
    gs = pk.magc_blockstack_bwd(u, [par], dout, fs["l_ckpt"], fs["ssm_ckpt"], fs["conv_ckpt"], H, P, G, N, Q, seg, 1)["grads"][0]
    assert torch.equal(fs["ssm_ckpt"][0, 1:], f["ssm_ckpt"][1:]) and torch.equal(fs["conv_ckpt"][0, 1:], f["conv_ckpt"][1:])
    for k in GRADS:
        assert torch.equal(gs[k], g[k]), k


@pytest.mark.parametrize("case", [
    # H, segment, L
    (80, 4096, 8192),
    (64, 1024, 10240),
])
def test_score_gradients_of_a_stack_are_rounded_once(case):
    """2-norm error of the gradients of B and C against 64 bits, read off the gradient of the input: the first columns of the input
    are B and C and nothing else, the convolution passes its last input on, and the output projection leaves those columns alone, so
    that nothing is added to their gradients.  The scan's own bar is 1.58 r, r = 1.66e-3 the root mean square of a rounding to bf16
    (test_gpu_slices.py, which derives it); behind it the gradient passes through SiLU and is rounded once more: (1.58^2 + 1)^1/2 r
    = 1.87 r.  Partial sums in bf16 add another r: (3 + 1)^1/2 r = 2 r and more."""
    H, seg, L = case
    P, G, N, Q, dm = 64, 1, 128, 256, 32 * H
    d_inner, conv_dim, _ = block_ref.dims(None, H, P, G, N)
    d = draw(92, L, dm, H, P, G, N)
    p, bc = d["p"], slice(2 * d_inner, d_inner + conv_dim)
    p["W_in"][:, :2 * N], p["W_in"][bc], p["W_out"][:2 * N] = 0.0, 0.0, 0.0
    p["W_in"][bc, :2 * N] = np.eye(2 * N)
    p["conv_w"], p["conv_b"] = np.tile([0.0, 0.0, 0.0, 1.0], (conv_dim, 1)), np.zeros(conv_dim)
    d["u"][:, :2 * N] = BF(d["u"][:, :2 * N] / np.sqrt(N))
    d["dout"][:, :2 * N] = 0.0
    x0, dout, par = dev_bf16(d["u"]), dev_bf16(d["dout"]), to_dev(p)
    f = pk.magc_blockstack_fwd(x0, [par], H, P, G, N, Q, seg, 1)
    got = host(pk.magc_blockstack_bwd(x0, [par], dout, f["l_ckpt"], f["ssm_ckpt"], f["conv_ckpt"], H, P, G, N, Q, seg, 1)["dx0"])[:, :2 * N]
    # in 64 bits from the tensors that the scan reads, each rounded as it is stored
    st = lambda v: np.asarray(synth.round_bf16(v), dtype=np.float64)  # noqa: E731
    fo = block_ref.block_fwd(d["u"], p, H, P, G, N, 1e-5, store=synth.round_bf16)
    z, y, xBC = fo["zxbcdt"][:, :d_inner], fo["y"], fo["xBC"]
    dy = st(norm_ref.gated_rmsnorm_bwd(y, z, p["norm_w"], st(d["dout"] @ p["W_out"]), 1e-5, G)["dy"])
    g = ssd_ref.ssd_bwd(xBC[:, :d_inner].reshape(1, L, H, P), fo["dt"][None], p["A"], xBC[None, :, None, d_inner:d_inner + N],
                        xBC[None, :, None, d_inner + N:], p["D"], dy.reshape(1, L, H, P))
    v = d["u"][:, :2 * N]
    sg = 1.0 / (1.0 + np.exp(-v))
    want = np.concatenate([g["dB"][0, :, 0], g["dC"][0, :, 0]], axis=1) * sg * (1.0 + v * (1.0 - sg))
    for k, cols in (("dB", slice(0, N)), ("dC", slice(N, 2 * N))):
        err = np.linalg.norm(got[:, cols] - want[:, cols]) / np.linalg.norm(want[:, cols])
        assert err < 1.87 * 1.66e-3, (k, err)
