"""The passes that walk the heads of a chunk ask for the next heads in pieces while they work on one: one, two, three and many
heads to a workgroup, at every chunk length, with a ragged last chunk; every gradient against the oracle."""
import numpy as np
import pytest

from paper_2411_19460_amd import synth
from parity_util import TOL, check, dev_inputs, host, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # Bt, L, H, G, Q, segment
    (1, 150 * 64 + 9, 1, 1, 64, 16384),     # 151 chunks: a head (and with more heads: all of them) to a workgroup
    (1, 150 * 64 + 9, 2, 1, 64, 16384),
    (1, 150 * 64 + 9, 3, 1, 64, 16384),
    (2, 70 * 64 + 1, 5, 1, 64, 8192),
    (1, 64 * 128 - 3, 5, 1, 128, 8192),
    (2, 40 * 128 - 127, 6, 2, 128, 8192),   # three heads to a group
    (1, 64 * 256 - 200, 2, 1, 256, 16384),
    (1, 64 * 256 - 200, 3, 1, 256, 16384),
    (1, 30 * 256 + 1, 9, 1, 256, 8192),
])
def test_heads_of_a_workgroup(case):
    Bt, L, H, G, Q, seg = case
    d = synth.make_layer_inputs(synth.SSDConfig("t", "bf16", Bt, L, H, 64, 128, G, 1, L, index=97), with_states=True)
    *_, g = run_gpu(dev_inputs(d, "bf16"), Q, seg)
    _, go = run_oracle(d)
    for k in ("dx", "ddt", "dB", "dC", "dD", "dinit_state"):
        check(k, host(g[k]), go[k], TOL["bf16"])
    # dA = sum over the tokens of dt (ddt - f) / A, f the direct part of ddt: over 10^4 tokens the terms cancel to a hundredth
    # of their size or less.  A token's term is off by TOL of its size at most, as ddt is, its sign independent of the others'.
    terms = np.asarray(d["dt"], np.float64) * go["ddt"] / np.asarray(d["A"], np.float64)
    bound = TOL["bf16"] * np.sqrt((terms ** 2).sum((0, 1)))
    err = np.abs(host(g["dA"]) - go["dA"])
    assert (err <= bound).all(), (err / bound).max()
