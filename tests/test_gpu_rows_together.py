"""The forward passes of a stack walk several segments as one set of launches (block.hip: plan_pass), and a long prompt in equal
pieces.  Neither the result nor the checkpoints may depend on it: sequences just longer than what may be walked together, against
one segment for the whole sequence, and the checkpoints against the states that inference leaves behind the same tokens.  The
backward pass walks the caller's segments."""
import pytest
import torch

import paper_2411_19460_amd as pk
from test_gpu_block import dev_bf16, draw, to_dev

pytestmark = pytest.mark.gpu


def _layers(n, dm, H, P, G, N):
    return [to_dev(draw(70 + j, 1, dm, H, P, G, N, True)["p"]) for j in range(n)]


def _input(L, dm, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn((L, dm), generator=g, device="cuda", dtype=torch.bfloat16)


def _close(a, b, band, what):
    err, top = float((a.float() - b.float()).abs().max()), float(b.float().abs().max())
    assert err <= band * top, (what, err, top)


@pytest.mark.parametrize("case", [
    # d_model, H, P, G, N, chunk, segment, L, layers, interval, segments looked at
    (128, 8, 64, 1, 128, 128, 1024, 70000, 2, 1, (1, 64, 65, 68)),     # 65 segments walked together, then four and a short one
    (128, 8, 64, 2, 128, 256, 33792, 70001, 2, 2, (1, 2)),             # one segment and a short one: two of them are too many
    (64, 8, 16, 1, 16, 2, 2, 37, 1, 1, (1, 2, 18)),                    # segments shorter than the convolution's window
])
def test_segments_walked_together(case):
    dm, H, P, G, N, Q, seg, L, NL, l, slots = case
    layers, x0, dout = _layers(NL, dm, H, P, G, N), _input(L, dm, 1), _input(L, dm, 2)
    run = lambda s: pk.magc_blockstack_fwd(x0, layers, H, P, G, N, Q, s, l)  # noqa: E731
    back = lambda s, f: pk.magc_blockstack_bwd(x0, layers, dout, f["l_ckpt"], f["ssm_ckpt"], f["conv_ckpt"], H, P, G, N, Q, s, l)  # noqa: E731
    whole = -(-L // seg) * seg
    f, f1 = run(seg), run(whole)
    assert torch.equal(f["out"], f1["out"])
    g, g1 = back(seg, f), back(whole, f1)
    # the bands of the grid's own tests: an adjoint of a state is rounded to bf16 where the cut is
    _close(g["dx0"], g1["dx0"], 2.0 ** -6, "dx0")
    for j in range(NL):
        for k in g["grads"][j]:
            _close(g["grads"][j][k], g1["grads"][j][k], 2.0 ** -6, (j, k))
    for k in slots:
        st = pk.magc_blockstack_infer(x0[:k * seg].contiguous(), layers, H, P, G, N, Q, seg)
        for j in range(NL):
            _close(f["ssm_ckpt"][j, k], st["ssm_state"][j], 2.0 ** -7, ("ssm", j, k))
            _close(f["conv_ckpt"][j, k], st["conv_state"][j], 2.0 ** -7, ("conv", j, k))


def test_a_long_prompt_in_equal_passes():
    dm, H, P, G, N, Q, seg, L = 128, 8, 64, 1, 128, 128, 4096, 140001      # two passes of at most 70016 tokens
    layers, x0 = _layers(2, dm, H, P, G, N), _input(L, dm, 3)
    st = pk.magc_blockstack_infer(x0, layers, H, P, G, N, Q, seg)
    a = pk.magc_blockstack_infer(x0[:40000].contiguous(), layers, H, P, G, N, Q, seg)
    b = pk.magc_blockstack_infer(x0[40000:].contiguous(), layers, H, P, G, N, Q, seg, ssm_state=a["ssm_state"], conv_state=a["conv_state"])
    _close(st["out"], torch.cat([a["out"], b["out"]]), 2.0 ** -6, "out")
    _close(st["ssm_state"], b["ssm_state"], 2.0 ** -6, "ssm")
    _close(st["conv_state"], b["conv_state"], 2.0 ** -6, "conv")
    f = pk.magc_blockstack_fwd(x0, layers, H, P, G, N, Q, seg, 1)
    assert torch.equal(f["out"], st["out"])
