"""The chunk-state launch forms the decay weights of its heads eight at a time: slices of more than eight heads, of no multiple of
eight, with packed sequences, and an odd number of score blocks.  Every tensor against the oracle."""
import numpy as np
import pytest
import torch

from oracle import ssd_ref
from paper_2411_19460_amd import synth
from parity_util import TOL, check, dev_inputs, host
from test_gpu_slices import test_slices_of_a_launch_on_its_own as check_slices
import paper_2411_19460_amd as pk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # Bt, L, H, G, Q, segment
    (1, 140 * 64 - 3, 19, 1, 64, 8960),      # 19 heads a workgroup: eight, eight, three
    (1, 150 * 128 - 5, 11, 1, 128, 19200),   # eight and three
    (1, 130 * 256 - 1, 17, 1, 256, 33280),   # eight, eight, one
    (1, 7 * 64, 8, 1, 64, 448),              # seven score blocks, two a workgroup
])
def test_slices_of_many_heads(case):
    check_slices(case)


def test_packed_sequences_in_slices_of_many_heads():
    Bt, L, H, G, Q = 1, 140 * 64 - 3, 19, 1, 64
    d = synth.make_layer_inputs(synth.SSDConfig("t", "bf16", Bt, L, H, 64, 128, G, 1, L, index=98))
    reset = np.zeros((Bt, L), np.uint8)
    reset[:, ::611] = 1
    dv = dev_inputs(d, "bf16")
    y, fin, _ = pk.ssd_fwd(dv["x"], dv["dt"], dv["A"], dv["B"], dv["C"], dv["D"], Q, 8960, seq_reset=torch.from_numpy(reset).cuda())
    cuts = list(range(0, L, 611)) + [L]
    parts = [ssd_ref.ssd_fwd(*(np.ascontiguousarray(d[k][:, a:b]) if k in ("x", "dt", "B", "C") else d[k] for k in ("x", "dt", "A", "B", "C", "D")), None, b - a)
             for a, b in zip(cuts, cuts[1:])]
    check("y", host(y), np.concatenate([p["y"] for p in parts], axis=1), TOL["bf16"])
    check("final_state", host(fin), parts[-1]["final_state"], TOL["bf16"])
