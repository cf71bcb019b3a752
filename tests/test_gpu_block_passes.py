"""What a stack of blocks joins into one pass, or leaves out, against the blocks called one by one: the residual with the next
layer's normalisation, the gradient round a block, states replaced in place, gradients stored by the first segment of a call
instead of cleared and added to."""
import numpy as np
import pytest
import torch

import paper_2411_19460_amd as pk
from parity_util import TOL, check, host
from test_gpu_block import GRADS, dev_bf16, draw, to_dev

pytestmark = pytest.mark.gpu

H, P, G, N, Q = 8, 64, 1, 128, 128
WIDTHS = [128, 1000, 16392]  # one vector a lane; a last vector that is no lane's; wider than a row of the joined pass


def stack(dm, L, NL=3, pre=True):
    d = [draw(80 + j, L, dm, H, P, G, N, pre) for j in range(NL)]
    return dev_bf16(d[0]["u"]), dev_bf16(d[0]["dout"]), [to_dev(q["p"]) for q in d]


@pytest.mark.parametrize("dm", WIDTHS)
@pytest.mark.parametrize("L", [17, 300])
def test_prompt_equals_the_blocks_one_by_one(dm, L):
    x, _, layers = stack(dm, L)
    r = pk.magc_blockstack_infer(x, layers, H, P, G, N, Q, 128)
    for j, p in enumerate(layers):
        f = pk.magc_block_fwd(x, p, H, P, G, N, Q, 128, checkpoints=False)
        x = (x.float() + f["out"].float()).to(torch.bfloat16)
        check(f"layer {j} ssm state", host(r["ssm_state"][j]), host(f["final_ssm"]), TOL["bf16"])
        check(f"layer {j} conv state", host(r["conv_state"][j]), host(f["final_conv"]), TOL["bf16"])
    check("out", host(r["out"]), host(x), TOL["bf16"])


@pytest.mark.parametrize("dm", WIDTHS)
def test_backward_equals_the_blocks_one_by_one(dm):
    x, dout, layers = stack(dm, 300, 2)
    f = pk.magc_blockstack_fwd(x, layers, H, P, G, N, Q, 128, 2)
    b = pk.magc_blockstack_bwd(x, layers, dout, f["l_ckpt"], f["ssm_ckpt"], f["conv_ckpt"], H, P, G, N, Q, 128, 2)
    one = pk.magc_block_fwd(x, layers[0], H, P, G, N, Q, 128)
    two_in = (x.float() + one["out"].float()).to(torch.bfloat16)
    two = pk.magc_block_fwd(two_in, layers[1], H, P, G, N, Q, 128)
    d = dout
    for j, u, q in ((1, two_in, two), (0, x, one)):
        g = pk.magc_block_bwd(u, layers[j], d, q["ssm_ckpt"], q["conv_ckpt"], H, P, G, N, Q, 128)
        d = (d.float() + g["du"].float()).to(torch.bfloat16)
        for k in GRADS + ("dpre_norm_w",):
            check(f"layer {j} {k}", host(b["grads"][j][k]), host(g[k]), TOL["bf16"])
    check("dx0", host(b["dx0"]), host(d), TOL["bf16"])


def test_gradients_are_stored_added_to_and_shared():
    """Buffers that hold NaN; the flag that adds to what they hold; layers that share their buffers (the sum of the layers').
    A sum of 2 or 3 fp32 values in another order differs by rounding: 1e-5 of the largest covers some 100 of them."""
    x, dout, layers = stack(128, 300)
    f = pk.magc_blockstack_fwd(x, layers, H, P, G, N, Q, 128, 2)
    run = lambda **kw: pk.magc_blockstack_bwd(x, layers, dout, f["l_ckpt"], f["ssm_ckpt"], f["conv_ckpt"], H, P, G, N, Q, 128, 2, **kw)["grads"]  # noqa: E731
    filled = lambda v: {k: torch.full_like(t, v) for k, t in want[0].items()}  # noqa: E731
    want = run()
    got = run(grads=[filled(float("nan")) for _ in layers])
    tied = filled(float("nan"))
    run(grads=[tied] * len(layers))
    part = [filled(float("nan")) for _ in layers]
    part[2]["dW_out"] = part[0]["dW_out"]
    run(grads=part)
    twice = run(grads=[{k: t.clone() for k, t in g.items()} for g in want], flags=pk.SSD_FLAG_ACCUM_PARAM)
    for k in want[0]:
        for j in range(len(layers)):
            assert torch.equal(got[j][k], want[j][k]), (j, k)
            check(f"layer {j} {k} added", host(twice[j][k]), 2 * host(want[j][k]), 1e-5)
        check(f"{k} shared", host(tied[k]), sum(host(g[k]) for g in want), 1e-5)
    check("dW_out of two layers", host(part[0]["dW_out"]), host(want[0]["dW_out"]) + host(want[2]["dW_out"]), 1e-5)
    assert torch.equal(part[1]["dW_out"], want[1]["dW_out"]) and torch.equal(part[0]["dW_in"], want[0]["dW_in"])


def test_gradients_of_no_tokens_are_zero():
    x, dout, layers = stack(128, 1, 1)
    nan = {k: torch.full_like(t, float("nan"), dtype=torch.float32) for k, t in (("d" + n, t) for n, t in layers[0].items())}
    e = x[:0].contiguous()
    pk.magc_blockstack_bwd(e, layers, e, None, None, None, H, P, G, N, Q, 128, 1, grads=[nan])
    assert all(np.all(host(t) == 0) for t in nan.values())
