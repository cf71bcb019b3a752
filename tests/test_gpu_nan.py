"""A NaN in an input reaches every output that depends on it: what the recurrence, token by token, makes NaN never comes out of
the chunked kernels as a number."""
import numpy as np
import pytest
import torch

import paper_2411_19460_amd as pk
from paper_2411_19460_amd import synth
from parity_util import dev_inputs, host, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["x", "dt", "B", "C", "dy"])
@pytest.mark.parametrize("case", [
    # dtype, P, N, Q, flags
    ("f32", 16, 24, 256, 0),                                   # four tiles of 64 tokens in a chunk
    ("bf16", 64, 128, 256, pk.SSD_FLAG_GENERIC_KERNELS),
    ("bf16", 64, 128, 256, 0),
])
def test_nan_is_not_lost(case, where):
    dtype, P, N, Q, flags = case
    d = synth.make_layer_inputs(synth.SSDConfig("t", dtype, 1, 512, 2, P, N, 1, 1, 512, index=92), with_states=True)
    d[where][0, 200] = np.nan
    y, fin, _, g = run_gpu(dev_inputs(d, dtype), Q, 512, flags)
    f, go = run_oracle(d, None)
    for name, got, want in [("y", y, f["y"]), ("final_state", fin, f["final_state"])] + [(k, g[k], go[k]) for k in ("dx", "ddt", "dA", "dB", "dC", "dD", "dinit_state")]:
        lost = np.isnan(want) & ~np.isnan(host(got))
        assert not lost.any(), f"{name}: {lost.sum()} of {np.isnan(want).sum()} NaN came out as numbers"


@pytest.mark.parametrize("Q", [64, 128, 256])
def test_an_infinity_in_the_last_token_of_a_ragged_chunk_stays_one(Q):
    """The rows a ragged last chunk lacks contribute nothing: an infinite B (C) of the last token makes its column of the state
    (of the initial state's gradient) an infinity with the sign of x (of dy), as token by token, and leaves the other columns
    alone."""
    L, n = 300, 5
    d = synth.make_layer_inputs(synth.SSDConfig("t", "bf16", 1, L, 1, 64, 128, 1, 1, L, index=93), with_states=True)
    d["A"][:] = -0.5                                           # nothing decays to zero on the way (0 inf = NaN)
    for k, vec, out in (("B", "x", "final_state"), ("C", "dy", "dinit_state")):
        e = {**d, k: d[k].copy()}
        e[k][0, -1, 0, n] = np.inf
        _, fin, _, g = run_gpu(dev_inputs(e, "bf16"), Q, None)
        got = host(fin if out == "final_state" else g[out])[0, 0]
        assert np.array_equal(got[:, n], np.sign(e[vec][0, -1, 0]) * np.inf), f"{out}: {got[:4, n]}"
        assert np.isfinite(np.delete(got, n, axis=1)).all(), out
        if k == "C":                                           # dB of the last chunk: dG[last, j] C[last]
            lost = np.isnan(host(g["dB"])[0, L - L % Q:, 0])
            assert not lost.any(), f"dB: {lost.sum()} NaN"
