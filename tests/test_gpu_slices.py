"""Head slices of the launches that have the machine to themselves: spans whose passes are cut into slices of different
length (workgroups of one round), or whose forward launches leave the general rule, every tensor against the oracle."""
import numpy as np
import pytest

from parity_util import TOL, check, dev_inputs, host, run_gpu, run_oracle
from paper_2411_19460_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # Bt, L, H, G, Q, segment
    (1, 16 * 256 - 7, 80, 1, 256, 4096),   # 16 chunks: five slices of dx and dG, two of the head sums
    (1, 3 * 256 + 5, 24, 1, 256, 1024),    # a slice per head beside slices of three
    (2, 4 * 256, 24, 2, 256, 512),         # two batches, two groups
    (1, 31 * 256 + 1, 24, 1, 256, 2048),   # one slice of the head sums
    (1, 40 * 256 - 200, 10, 1, 256, 4096),  # forward slices of two heads
    (2, 3001, 14, 2, 128, 1024),           # chunks of 128: two workgroups of a forward launch on a compute unit
    (1, 4000, 80, 1, 64, 4096),            # chunks of 64: eight slices where the general rule takes five
    (2, 2500, 18, 2, 64, 4096),            # chunk states and adjoints in three where it takes one
])
def test_slices_of_a_launch_on_its_own(case):
    Bt, L, H, G, Q, seg = case
    d = synth.make_layer_inputs(synth.SSDConfig("t", "bf16", Bt, L, H, 64, 128, G, 1, L, index=97), with_states=True)
    y, fin, _, g = run_gpu(dev_inputs(d, "bf16"), Q, seg)
    f, go = run_oracle(d)
    check("y", host(y), f["y"], TOL["bf16"])
    check("final_state", host(fin), f["final_state"], TOL["bf16"])
    for k in ("dx", "ddt", "dA", "dB", "dC", "dD", "dinit_state"):
        check(k, host(g[k]), go[k], TOL["bf16"])


@pytest.mark.parametrize("case", [
    # Bt, L, H, G, Q, segment
    (1, 32 * 256, 24, 1, 256, 2048),       # 32 chunks: three slices
    (1, 16 * 256 - 7, 80, 1, 256, 4096),   # 16: five
    (2, 8 * 256, 24, 2, 256, 1024),        # two batches, two groups
    (1, 16 * 128, 80, 1, 128, 1024),       # chunks of 128: more slices than half of the general rule's
    (1, 5000, 24, 1, 128, 2048),           # the same in a span shorter than its whole segments
    (1, 61 * 256 + 9, 64, 1, 256, 4096),   # a span of more units than lanes take
])
def test_few_slices_round_the_score_gradients_once(case):
    """2-norm error of dB and dC.  A number stored in bf16 is off by r = 1.66e-3 in the root mean square (uniform within half
    a unit, averaged over the mantissas).  dB is rounded where it is stored (r); of its two parts the score gradients are
    rounded on their way to the matrix core (r), the head sums, a share v of the square of the whole, have two rounded operands
    (2^1/2 r): (2 + v)^1/2 r in all.  A state decays by a factor e within 33 tokens of the mean step size even at A = -1, so
    less than half of what reaches a token comes from other chunks: v < 1/2, 1.58 r = 2.62e-3.  Partial sums of the score
    gradients in bf16 add another r: more than 3^1/2 r = 2.87e-3."""
    Bt, L, H, G, Q, seg = case
    d = synth.make_layer_inputs(synth.SSDConfig("t", "bf16", Bt, L, H, 64, 128, G, 1, L, index=101))
    _, _, _, g = run_gpu(dev_inputs(d, "bf16"), Q, seg)
    _, go = run_oracle(d)
    for k in ("dB", "dC"):
        err = np.linalg.norm(host(g[k]) - go[k]) / np.linalg.norm(go[k])
        assert err < 1.58 * 1.66e-3, (k, err)
