"""The in-LDS pass of the most-significant-digit calibration at the edges of
its 8,192-record tiles, against the oracle: sub-buckets (here one source each)
just below, at and just above one tile, pairs that fill a tile exactly or
miss by one, and tiles that straddle two 2^16-connection blocks.  Targets,
delays and indices are whole numbers and must be equal; weights within the
oracle's bound (parity.check_calibrated)."""
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


@pytest.mark.parametrize("k", [4095, 4096, 4097, 8191, 8192, 8193, 16385])
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
