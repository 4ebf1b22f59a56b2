"""The queued Connect calls of contexts calibrated together, generated in one
launch: what each context's timing reports of it, and a first context without
arena room for all calls' descriptors."""
import pytest

import oracle
from paper_2306_09855_amd import workloads as W
from parity import check_calibrated

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2306_09855_amd import ng  # noqa: E402
from paper_2306_09855_amd.network import Network, arena_bytes_for, calibrate_many  # noqa: E402

B = 1 << 16
W_D = (("normal", 0.5, 0.05), ("uniform_int", 1, 30))


def _workloads(calls, each, count):
    return [W.Workload("queued", 40 + k, [700],
                       [W.Call("fixed_total_number", (i % 500, 200), (i % 300, 400), each + k, *W_D)
                        for i in range(calls)]) for k in range(count)]


def _queued(wl, arena=None):
    net = Network(wl.seed, wl.h, B, arena or arena_bytes_for(wl.n_syn, wl.n_nodes, wl.max_delay, B))
    ng.ng_set_schedule(net.ctx, {**ng.ng_get_schedule(net.ctx), "queued_calls": 4096})
    return net.build(wl, calibrate=False)


def _check(net, wl):
    ref = oracle.build_network(wl.seed, wl.h, wl.n_nodes, wl.calls)
    check_calibrated(net.fetch(), *net.group_index(), ref, wl.calls)


@pytest.mark.parametrize("timed", [(0, 1, 2), (0,), (1,), (0, 2)])
def test_each_context_times_its_own_generation(timed):
    wls = _workloads(8, 1000, 3)
    nets = [_queued(wl) for wl in wls]
    try:
        for k in timed:
            ng.ng_enable_timing(nets[k].ctx, True)
        calibrate_many(nets)
        for k, (net, wl) in enumerate(zip(nets, wls)):
            got = ng.ng_read_timing(net.ctx, reset=True, records=True)
            if k in timed:
                launches, ms, records = got["generate_batch"]
                assert launches == 1 and ms > 0 and records == wl.n_syn
            else:
                assert not got
            _check(net, wl)
    finally:
        for net in nets:
            net.close()


def test_no_room_for_the_descriptors_of_all_contexts():
    calls, count = 4000, 4  # at least 160 bytes a call: 2.5 MB in all
    wls = _workloads(calls, 2, count)
    upload = 160 * calls * count
    nets = [_queued(wl) for wl in wls]
    try:
        before = nets[0].memory_stats()[0]
        calibrate_many(nets)
        assert nets[0].memory_stats()[1] - before >= upload  # one upload, from the first context's arena
    finally:
        for net in nets:
            net.close()
    nets = [_queued(wl, before + upload - 4096 if k == 0 else None) for k, wl in enumerate(wls)]
    try:
        calibrate_many(nets)
        for net, wl in zip(nets, wls):
            _check(net, wl)
    finally:
        for net in nets:
            net.close()
