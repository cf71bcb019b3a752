"""The forward pass works in chunks of the caller's length, whatever segments the sequence is cut into and whichever entry point
runs it: the same bits with long segments of several chunks, with short ones, in one piece and from the static scratch."""
import pytest
import torch

import paper_2411_19460_amd as pk
from paper_2411_19460_amd import synth
from parity_util import dev_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk,packed", [(64, False), (128, False), (128, True)])
def test_results_do_not_depend_on_where_the_sequence_is_cut(chunk, packed):
    L, H = 3077, 4
    d = synth.make_layer_inputs(synth.SSDConfig("t", "bf16", 1, L, H, 64, 128, 1, 1, L, index=91), with_states=True)
    dv = dev_inputs(d, "bf16")
    ins = [dv[k] for k in ("x", "dt", "A", "B", "C", "D")]
    reset = None
    if packed:                       # sequences of 100 tokens
        reset = torch.zeros((1, L), dtype=torch.uint8, device="cuda")
        reset[:, ::100] = 1
    y, fin, bnd = pk.ssd_fwd(*ins, chunk, 1024, dv["init_state"], seq_reset=reset)
    for segment in (512, 2048, None):
        y2, fin2, bnd2 = pk.ssd_fwd(*ins, chunk, segment, dv["init_state"], seq_reset=reset)
        assert torch.equal(y, y2) and torch.equal(fin, fin2), segment
        if segment:
            for k in range(bnd2.shape[1]):
                if k * segment % 1024 == 0:
                    assert torch.equal(bnd2[:, k], bnd[:, k * segment // 1024])
    out = {"y": torch.empty_like(y), "final_state": torch.empty_like(fin), "boundary_states": torch.empty_like(bnd)}
    y3, fin3, bnd3 = pk.ssd_fwd_static(*ins, chunk, 1024, out, dv["init_state"], seq_reset=reset)
    torch.cuda.synchronize()
    assert torch.equal(y, y3) and torch.equal(fin, fin3) and torch.equal(bnd, bnd3)
