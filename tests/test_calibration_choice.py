"""Which form a calibration takes, from the plan queries (no device)."""
import pytest

import bench
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


@pytest.mark.parametrize("n,nodes,delay,form", [
    ((1 << 24) - 1, 20_000, 31, "lsd"),     # 2^24 connections
    (1 << 24, 20_000, 31, "msd"),
    (20_971_519, 1 << 18, 31, "lsd"),       # 2.5 per possible key: 2^18 nodes x 2^5 delays
    (20_971_520, 1 << 18, 31, "msd"),
    (30_000_000, 77_169, 30, "msd"),
    (445_000_000, 1_000_000, 63, "msd"),    # 6.95 per possible key
    (300_000_000, 77_169, 30, "msd"),
    (100_000, 2_000, 20, "lsd"),
    (2 ** 32 - 1, 77_169, 30, "lsd"),
    (300_000_000, 1 << 24, 31, "lsd"),      # keys of 29 bits
    (0, 100, 5, "lsd"),
])
def test_form_of_the_default_calibration(n, nodes, delay, form):
    assert ng.ng_calibration_form(n, nodes, delay) == form
    plan = ng.ng_calibration_plan(n, nodes, delay)["msd"]
    assert plan >= 1 if form == "msd" else plan <= 1


def test_form_refuses_what_the_plan_refuses():
    with pytest.raises(ng.NGError) as e:
        ng.ng_calibration_form(1000, 10, 0)
    assert e.value.status == ng.NG_ERR_INVALID_ARG
    assert ng.lib().ng_calibration_form(1000, 10, 1, 0, None) == ng.NG_ERR_INVALID_ARG


def test_bench_reports_the_form_that_ran():
    # between the plan's two bounds the default is the MSD form
    plan = ng.ng_calibration_plan(445_000_000, 1_000_000, 63)
    assert bench.calibrated_msd({"generate_batch": 1, "msd_scatter_a": 1, "scan": 1})
    assert not bench.calibrated_msd({"generate": 1, "upsweep": 1, "scan": 1, "downsweep": 1})
    assert bench.moved_bytes("msd_count_a", 445_000_000, plan) == 4.0 * 445_000_000
