"""Shape-generic kernels: rows of the head sums whose columns are not groups of four, one row or column past a tile, and
chunks whose last tile is ragged; every tensor against the oracle."""
import pytest

from paper_2411_19460_amd import synth
from parity_util import TOL, check, dev_inputs, host, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # dtype, Bt, L, H, P, G, N, Q, segment
    ("f32", 1, 130, 2, 3, 1, 33, 100, 200),      # columns one by one
    ("f32", 2, 65, 4, 65, 2, 66, 64, 64),        # one row past a tile, in every direction
    ("f32", 1, 191, 3, 64, 1, 68, 192, 192),     # groups of four that end inside a tile, three tiles of a chunk
    ("f32", 1, 257, 1, 1, 1, 1, 256, 512),       # a chunk of one token
    ("bf16", 1, 200, 8, 5, 1, 7, 72, 144),
])
def test_rows_and_columns_past_a_tile(case):
    dtype, Bt, L, H, P, G, N, Q, seg = case
    d = synth.make_layer_inputs(synth.SSDConfig("t", dtype, Bt, L, H, P, N, G, 1, L, index=99), with_states=True)
    y, fin, _, g = run_gpu(dev_inputs(d, dtype), Q, seg)
    f, go = run_oracle(d, None)
    check("y", host(y), f["y"], TOL[dtype])
    check("final_state", host(fin), f["final_state"], TOL[dtype])
    for k in ("dx", "ddt", "dA", "dB", "dC", "dD", "dinit_state"):
        check(k, host(g[k]), go[k], TOL[dtype])
