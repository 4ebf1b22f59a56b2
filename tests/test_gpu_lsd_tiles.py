"""The LSD calibration at the edges of its tile sizes and of its two ways to
turn counts into offsets: fewer and more records than one 2,048-record tile,
192 ranges (summed by the downsweep) and 193 (scanned), the last record count
with small tiles and the first with large ones, and several contexts in one
packed calibration.  Against the oracle where it is quick, else bit for bit
against the most-significant-digit form."""
import numpy as np
import pytest

import oracle
from paper_2306_09855_amd import workloads as W
from parity import check_calibrated

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2306_09855_amd.network import Network, arena_bytes_for, calibrate_many  # noqa: E402

W_D = (("normal", 0.5, 0.05), ("uniform_int", 1, 30))


def _wl(n, nodes, seed=3):
    return W.Workload("lsd_edges", seed, [nodes], [W.Call("fixed_total_number", (0, nodes), (0, nodes), n, *W_D)])


def _net(wl, block):
    return Network(wl.seed, wl.h, block, arena_bytes_for(wl.n_syn, wl.n_nodes, wl.max_delay, block))


def _sorted(wl, calibration, block):
    with _net(wl, block) as net:
        net.set_calibration(calibration)
        net.build(wl)
        return (net.fetch(), *net.group_index())


@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 192 * 2048, 192 * 2048 + 1])
@pytest.mark.parametrize("nodes", [40, 9_000])  # few large groups, and many small ones
def test_small_tiles(n, nodes):
    wl = _wl(n, nodes)
    ref = oracle.build_network(wl.seed, wl.h, nodes, wl.calls)
    out, gp, gs = _sorted(wl, "lsd", 1 << 16)
    check_calibrated(out, gp, gs, ref, wl.calls)


def _on_device(wl, calibration, block):
    with _net(wl, block) as net:
        net.set_calibration(calibration)
        net.build(wl)
        return (net.fetch(device=True), *net.group_index())


@pytest.mark.parametrize("n,block", [((1 << 23) + 1, 1 << 20), ((1 << 27) - 1, 1 << 24), (1 << 27, 1 << 24)])
def test_both_tile_sizes_equal_the_msd_form(n, block):
    wl = _wl(n, 30_000)
    a, b = _on_device(wl, "lsd", block), _on_device(wl, "msd", block)
    for k in ("src", "tgt", "delay"):
        assert torch.equal(a[0][k], b[0][k]), k
    assert torch.equal(a[0]["w"].view(torch.int32), b[0]["w"].view(torch.int32))
    assert np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])


@pytest.mark.parametrize("sizes", [(1, 2049, 0, 300_000), (500_000, 3, 192 * 2048)])
def test_packed_contexts(sizes):
    wls = [_wl(n, 700, seed=20 + k) for k, n in enumerate(sizes)]
    nets = [_net(wl, 1 << 16) for wl in wls]
    try:
        for net, wl in zip(nets, wls):
            net.build(wl, calibrate=False)
        calibrate_many(nets)
        for net, wl in zip(nets, wls):
            ref = oracle.build_network(wl.seed, wl.h, wl.n_nodes, wl.calls)
            check_calibrated(net.fetch(), *net.group_index(), ref, wl.calls)
    finally:
        for net in nets:
            net.close()
