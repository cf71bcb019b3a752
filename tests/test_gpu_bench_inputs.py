"""What the benchmark's line is made from besides its own timings is there where it runs."""
import pytest

import bench

pytestmark = pytest.mark.gpu


def test_measured_traffic_of_the_dominant_kernel_is_found():
    """The HBM bytes per launch of the headline's dominant kernel, from the counter runs kept in the tree (an unreadable file
    reads as "not measured")."""
    assert bench.measured_traffic("mfma_bwd_trio", "c2_2p7b_64k_bf16") > 0
