"""Head slices of the launches that have the machine to themselves: spans whose passes are cut into slices of different
length (workgroups of one round), or whose forward launches leave the general rule, every tensor against the oracle."""
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
