"""Head slices of two lengths one apart (the slices need not divide the heads of a group): every tensor against the oracle."""
import pytest

from test_gpu_slices import test_few_slices_round_the_score_gradients_once as check_rounding
from test_gpu_slices import test_slices_of_a_launch_on_its_own as check_slices

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # Bt, L, H, G, Q, segment
    (1, 3333, 64, 1, 256, 4096),       # 14 chunks: slices of three and four heads forward, six and seven for dx and dG
    (1, 32 * 256 - 9, 23, 1, 256, 8192),  # a prime number of heads
    (2, 2000, 22, 2, 256, 2048),       # eleven heads a group
    (1, 3001, 13, 1, 128, 1024),
    (1, 2000, 7, 1, 64, 2048),
])
def test_slices_of_two_lengths(case):
    check_slices(case)


@pytest.mark.parametrize("case", [(1, 3333, 64, 1, 256, 4096), (1, 32 * 256 - 9, 23, 1, 256, 8192)])
def test_their_partial_sums_are_rounded_once(case):
    check_rounding(case)


@pytest.mark.parametrize("case", [
    # Bt, L, H, G, Q, segment
    (1, 15 * 128, 24, 1, 128, 4096),   # twelve slices, as many as the general rule's, where eight are no longer in the launch
    (1, 23 * 128, 8, 1, 128, 1024),    # a slice for every head
    (1, 31 * 256, 48, 1, 256, 4096),   # one round that ends with the general rule's launch
])
def test_one_round_keeps_its_partial_sums_in_fp32(case):
    check_rounding(case)


@pytest.mark.parametrize("case", [
    # Bt, L, H, G, Q, segment
    (1, 100, 37, 1, 128, 128),         # one chunk: a slice for every head, the last one on its own behind nine fours
    (1, 200, 6, 1, 256, 256),          # two behind one four
    (1, 60, 22, 2, 64, 64),            # eleven a group: three
    (1, 100, 8, 1, 128, 128),          # two fours
])
def test_a_slice_for_every_head_of_one_chunk(case):
    check_slices(case)
