"""One generation step for a few sequences at the sizes where its kernels change: two rows (vector ALUs) and three (matrix
cores), widths that are no multiple of a 256-wide piece, two groups whose norms scale the pieces, state rows of more than
128 columns, more rows per wave with more sequences.  Checked against the oracle run on each sequence alone."""
import pytest
import torch

import paper_2411_19460_amd as pk
from test_gpu_block import test_stack_generation_for_several_sequences_at_once as check_generation

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    # d_model, H, P, G, N, Q, pre-norm, sequences
    (128, 8, 64, 1, 128, 128, True, 2),
    (320, 8, 64, 1, 128, 128, True, 3),
    (768, 24, 64, 2, 128, 128, True, 12),
    (128, 8, 64, 1, 136, 64, True, 4),
])
def test_generation_rows(shape):
    check_generation(shape)


def test_parameters_are_checked_on_every_step():
    """A stack that one step accepted is refused once one of its tensors, at the same address, has another shape."""
    from paper_2411_19460_amd import binding
    want = binding._block_layout(torch.empty((1, 128), dtype=torch.bfloat16, device="cuda"), {}, 8, 64, 1, 128, 64, None, 1e-5)[1]
    layers = [{k: torch.zeros(shp, dtype=dty, device="cuda") for k, (shp, dty) in want.items()} for _ in range(2)]
    x = torch.zeros((1, 128), dtype=torch.bfloat16, device="cuda")
    step = lambda: pk.magc_blockstack_infer(x, layers, 8, 64, 1, 128, 64, 64)  # noqa: E731
    step()
    for k in ("W_in", "conv_w", "D"):
        t = layers[1][k]
        layers[1][k].unsqueeze_(0)
        with pytest.raises(ValueError, match=k):
            step()
        t.squeeze_(0)
    step()
    torch.cuda.synchronize()
