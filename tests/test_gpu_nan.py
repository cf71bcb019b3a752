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
