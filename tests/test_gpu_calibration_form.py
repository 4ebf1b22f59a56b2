"""The form that ng_calibration_form names is the one whose kernels the default
calibration launches, at its bounds and between them and the plan query's."""
import pytest

from paper_2306_09855_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2306_09855_amd import ng  # noqa: E402
from paper_2306_09855_amd.network import Network, arena_bytes_for  # noqa: E402


@pytest.mark.parametrize("n,nodes,delay", [
    ((1 << 24) - 1, 20_000, 31), (1 << 24, 20_000, 31), (20_971_519, 1 << 18, 31), (20_971_520, 1 << 18, 31),
    (1 << 25, 1 << 17, 31), (100_000, 2_000, 20)])
def test_kernels_are_those_of_the_named_form(n, nodes, delay):
    block = 1 << 22
    wl = W.Workload("form", 5, [nodes], [W.Call("fixed_total_number", (0, nodes), (0, nodes), n,
                                                ("normal", 0.5, 0.05), ("uniform_int", 1, delay))])
    with Network(wl.seed, wl.h, block, arena_bytes_for(n, nodes, delay, block)) as net:
        net.build(wl, calibrate=False)
        ng.ng_enable_timing(net.ctx, True)
        net.calibrate()
        names = set(ng.ng_read_timing(net.ctx, reset=True))
    form = ng.ng_calibration_form(n, nodes, delay)
    assert ("msd_tiles_c" in names) == (form == "msd") and ("downsweep" in names) == (form == "lsd")
