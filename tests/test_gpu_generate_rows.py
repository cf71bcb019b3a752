"""One generation step for a few sequences at the sizes where its kernels change: two rows (vector ALUs) and three (matrix
cores), widths that are no multiple of a 256-wide piece, two groups whose norms scale the pieces, state rows of more than
128 columns, more rows per wave with more sequences.  Checked against the oracle run on each sequence alone."""
import pytest

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
