"""GPU parity of the COPASS partition search at its dispatch edges: 32, 64,
128, 256 and 512 subarrays and one more (one to eight subarrays per lane, 64
samples of each up to 256, the bisection from 513 on), with a ragged last block,
blocks whose sources do not overlap, blocks that hold every source, and keys
shared by many thousand connections (exact counts where samples do not
narrow).  The COPASS arrays must be those of the LSD radix form bit for bit."""
import numpy as np
import pytest

from paper_2306_09855_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2306_09855_amd.network import Network, arena_bytes_for  # noqa: E402

B = 1 << 16


def _run(wl, mode, radix_bits=9):
    with Network(wl.seed, wl.h, B, arena_bytes_for(wl.n_syn, wl.n_nodes, wl.max_delay, B)) as net:
        net.set_calibration(mode)
        net.tune(radix_bits, 1024)
        net.build(wl)
        out = net.fetch(device=True)
        gp, gs = net.group_index()
    return out, gp, gs


def _same(x, y):
    (a, gpa, gsa), (b, gpb, gsb) = x, y
    for key in ("src", "tgt", "delay"):
        assert torch.equal(a[key], b[key]), key
    assert torch.equal(a["w"].view(torch.int32), b["w"].view(torch.int32))
    assert np.array_equal(gpa, gpb) and np.array_equal(gsa, gsb)


@pytest.mark.parametrize("blocks", [2, 32, 33, 64, 65, 128, 129, 256, 257, 512, 513])
def test_partition_search_sizes(blocks):
    n = (blocks - 1) * B + 4321
    pops = [5000, 3000]
    w = ("normal", 0.5, 0.05)
    calls = [
        # a third: every source in every block
        W.Call("fixed_total_number", (0, 8000), (5000, 3000), n // 3, w, ("uniform_int", 1, 20)),
        # a third: sources ascending over the blocks
        W.Call("fixed_outdegree", (0, 5000), (5000, 3000), n // 3 // 5000, w, ("uniform_int", 1, 20)),
        # two sources and one delay: two keys shared by the connections of many blocks
        W.Call("fixed_total_number", (4000, 2), (0, 8000), n // 6, w, ("const", 0.5)),
    ]
    rest = n - sum(c.n_syn() for c in calls)
    calls.append(W.Call("fixed_total_number", (0, 3000), (5000, 3000), rest, w, ("uniform_int", 1, 3)))
    wl = W.Workload("copass_search", 41 + blocks, pops, calls)
    assert -(-wl.n_syn // B) == blocks
    _same(_run(wl, "copass"), _run(wl, "lsd"))


@pytest.mark.parametrize("nodes,radix_bits", [(20, 9), (20, 4), (20, 5), (9000, 6), (9000, 4)])
def test_block_sort_passes(nodes, radix_bits):
    # 8-bit keys in one and two passes, 17-bit keys in three and five: a block
    # is sorted from itself unless one pass has to do
    n = 3 * B + 77
    wl = W.Workload("copass_passes", 5, [nodes],
                    [W.Call("fixed_total_number", (0, nodes), (0, nodes), n, ("normal", 0.5, 0.05),
                            ("uniform_int", 1, 7))])
    _same(_run(wl, "copass", radix_bits), _run(wl, "lsd"))
