"""The in-LDS pass of the most-significant-digit calibration at the edges of
its 8,192-record tiles, against the oracle: sub-buckets (here one source each)
just below, at and just above one tile, pairs that fill a tile exactly or
miss by one, tiles that straddle two 2^16-connection blocks, and larger
sub-buckets in one, two and three pieces of 16,384 records.  Targets,
delays and indices are whole numbers and must be equal; weights within the
oracle's bound (parity.check_calibrated)."""
import numpy as np
import pytest

import oracle
from paper_2306_09855_amd import workloads as W
from parity import check_calibrated

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2306_09855_amd import ng  # noqa: E402
from paper_2306_09855_amd.network import Network, arena_bytes_for  # noqa: E402

W_D = (("normal", 0.5, 0.05), ("const", 0.1))


@pytest.mark.parametrize("k", [4095, 4096, 4097, 8191, 8192, 8193, 16384, 16385, 40_000])
def test_sub_buckets_around_one_tile(k):
    n = 64
    calls = [W.Call("fixed_outdegree", (0, n // 2), (0, n), k, *W_D),
             W.Call("fixed_outdegree", (n // 2, n // 2), (0, n), 4096, *W_D)]
    wl = W.Workload("tile_edges", 11, [n], calls)
    plan = ng.ng_calibration_plan(wl.n_syn, n, 1, 1024)
    assert plan["msd"] >= 1 and plan["b3"] == 1 and plan["narrow_a"] == 1  # one source per sub-bucket, packed records
    ref = oracle.build_network(wl.seed, wl.h, n, calls)
    with Network(wl.seed, wl.h, 1 << 16, arena_bytes_for(wl.n_syn, n, 1, 1 << 16)) as net:
        net.set_calibration("msd")
        net.build(wl)
        out = net.fetch()
        gp, gs = net.group_index()
    check_calibrated(out, gp, gs, ref, calls)


def _arrays(wl, calibration, block):
    with Network(wl.seed, wl.h, block, arena_bytes_for(wl.n_syn, wl.n_nodes, wl.max_delay, block)) as net:
        net.set_calibration(calibration)
        net.build(wl, batched=True, calibrate=False)
        ng.ng_enable_timing(net.ctx, True)
        ng.ng_read_timing(net.ctx, reset=True)
        net.calibrate()
        names = set(ng.ng_read_timing(net.ctx, reset=True))
        return (net.fetch(), *net.group_index(), names)


def _same(a, b):
    for k in ("src", "tgt", "delay"):
        assert np.array_equal(a[0][k], b[0][k]), k
    assert np.array_equal(a[0]["w"].view(np.uint32), b[0]["w"].view(np.uint32))
    assert np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])


@pytest.mark.parametrize("n_calls,n_nodes,hi_exp", [(24, 300, 5.0), (40, 20_000, 5.0), (60, 200_000, 5.0)])
def test_uneven_sources_equal_the_lsd_form(n_calls, n_nodes, hi_exp):
    # from 50 connections per possible key to 0.1, with sources that hold
    # most of a call next to empty ones: the split of pass C by work, tiles
    # of few records spread over all waves, and listed sub-buckets in pieces
    wl = W.batch_mixed(n_calls=n_calls, n_nodes=n_nodes, hi_exp=hi_exp, gen_seed=8)
    a, b = _arrays(wl, "msd", 1 << 18), _arrays(wl, "lsd", 1 << 18)
    assert "msd_tiles_c" in a[3] and "downsweep" in b[3]
    _same(a, b)


def test_default_form_at_its_lower_bounds():
    # from 2^24 connections and 2.5 per possible key on the default is the
    # most-significant-digit form, below either bound the LSD form
    w, d = ("normal", 0.5, 0.05), ("uniform_int", 1, 31)
    n_dense = 20_000
    at = [((1 << 24) - 1, n_dense, False), (1 << 24, n_dense, True),
          (20_971_520, 1 << 18, True), (20_971_519, 1 << 18, False)]  # 2^18 nodes x 2^5 delays x 2.5
    for n, nodes, msd in at:
        wl = W.Workload("bounds", 5, [nodes], [W.Call("fixed_total_number", (0, nodes), (0, nodes), n, w, d)])
        got = _arrays(wl, "radix", 1 << 22)
        assert ("msd_tiles_c" in got[3]) == msd and ("downsweep" in got[3]) == (not msd), (n, nodes)
        if msd:
            _same(got, _arrays(wl, "lsd", 1 << 22))
