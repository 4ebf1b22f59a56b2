"""Which form a calibration takes, from the plan queries (no device)."""
import pytest

from paper_2306_09855_amd import build as B
from paper_2306_09855_amd import ng


@pytest.fixture(scope="module", autouse=True)
def built():
    import os
    if not os.path.exists(B.LIB):
        B.build()


@pytest.mark.parametrize("nodes,delay", [(77_169, 30), (200, 20), (1_000_000, 63)])
def test_msd_form_leaves_room_for_32_bit_steps(nodes, delay):
    # its kernels step up to 16,384 positions past the last record in 32 bits
    most = 2 ** 32 - 2 ** 15
    assert ng.ng_calibration_plan(most, nodes, delay)["msd"] >= 1
    for n in (most + 1, 2 ** 32 - 8191, 2 ** 32 - 1):
        assert not any(ng.ng_calibration_plan(n, nodes, delay).values()), n
