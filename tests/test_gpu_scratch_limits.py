"""What a calibration asks of its arena, and what it does when the arena does
not have it: results in arenas of just the size, bit for bit against an
ordinary build in the LSD form."""
import numpy as np
import pytest

from paper_2306_09855_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2306_09855_amd import ng  # noqa: E402
from paper_2306_09855_amd.network import Network, arena_bytes_for  # noqa: E402


def _up(nbytes):
    return max(256, -(-nbytes // 256) * 256)  # arena allocations come in 256 bytes


def _wl(n, nodes, delay):
    """n connections, a third of them from one source."""
    w, d = ("normal", 0.5, 0.05), ("uniform_int", 1, delay)
    return W.Workload("limits", 7, [nodes],
                      [W.Call("fixed_total_number", (nodes // 2, 1), (0, nodes), n // 3, w, d),
                       W.Call("fixed_total_number", (0, nodes), (0, nodes), n - n // 3, w, d)])


class _Built:
    """The workload's connections in an arena of `arena` bytes (None: ample),
    calibrated in `form`: arrays, index, kernels launched and arena bytes."""

    def __init__(self, wl, form, block, arena=None, calibrate=ng.ng_calibrate, ranges=1024):
        ample = arena_bytes_for(wl.n_syn, wl.n_nodes, wl.max_delay, block) + 24 * wl.n_syn
        with Network(wl.seed, wl.h, block, arena or ample) as net:
            net.set_calibration(form)
            net.tune(9, ranges)
            net.build(wl, calibrate=False)
            net.sync()
            self.before = net.memory_stats()[0]
            ng.ng_enable_timing(net.ctx, True)
            calibrate(net.ctx)
            self.kernels = set(ng.ng_read_timing(net.ctx, reset=True))
            _, self.peak, _ = net.memory_stats()
            self.arrays = net.fetch(device=True)
            self.index = net.group_index()

    def same(self, other):
        for k in ("src", "tgt", "delay"):
            assert torch.equal(self.arrays[k], other.arrays[k]), k
        assert torch.equal(self.arrays["w"].view(torch.int32), other.arrays["w"].view(torch.int32))
        assert np.array_equal(self.index[0], other.index[0]) and np.array_equal(self.index[1], other.index[1])


def _msd_bytes(n, nodes, delay, block, ranges=1024, digits=None):
    """The calibrated blocks, index and scratch of the most-significant-digit
    form: the records of each pass, a group slot per connection, the digit
    counts and tables, and a word per 10,241 connections for lists."""
    p = ng.ng_calibration_plan(n, nodes, delay, ranges)
    assert p["msd"] >= 1
    if digits:
        p["b1"], p["b2"], p["b3"] = digits
    rec_a, rec_b = (8 if p["narrow_a"] else 12), (8 if p["narrow_b"] else 12)
    nb, nsb = 1 << p["b1"], 1 << (p["b1"] + p["b2"])
    na = nb * -(-(-(-n // 10240)) // p["tpr"])
    nbc = (3 * ranges + nb) << p["b2"] if p["b2"] else 0
    scan = max(-(-x // 4096) + 1 for x in (na, nbc, nsb))
    split = min(max(-(-n // 61440), 1024), nsb)
    sizes = [4 * n] * (rec_a // 4 + (rec_b // 4 if p["b2"] else 1)) + [4 * na]
    sizes += [4 * nbc] if p["b2"] else []
    sizes += [4 * scan, 4 * (nb + 1), 4 * (nb + 1), 4 * nb, 4 * (nsb + 1), 4 * (nsb + 1),
              4 * nsb * max(1, (1 << p["b3"]) // 32), 4 * (split + 1), 4, 4 * (n // 10241 + 1),
              4 * (nodes + 1), 4 * (min(n, nodes * delay) + 1)]
    return sum(map(_up, sizes)) + -(-n // block) * 14 * block


@pytest.mark.parametrize("n,nodes,delay", [
    (5_000, 2_000, 7),           # less than one LDS load
    (2_000_001, 30_000, 31),     # two scatters, packed records, 9-bit last digit
    (3_000_000, 100, 3),         # one scatter
    (2_500_000, 1 << 24, 3),     # unpacked records
])
def test_msd_form_in_its_bytes(n, nodes, delay):
    block = 1 << 18
    wl = _wl(n, nodes, delay)
    need = _msd_bytes(n, nodes, delay, block)
    ample = _Built(wl, "msd", block)
    assert "msd_tiles_c" in ample.kernels
    assert ample.peak - ample.before <= need
    tight = _Built(wl, "msd", block, ample.before + need)
    lsd = _Built(wl, "lsd", block)
    assert "downsweep" in lsd.kernels
    ample.same(lsd)
    tight.same(lsd)


@pytest.mark.parametrize("n,nodes,delay,usual,wider", [
    (1_840_000, 800, 1, (5, 5, 1), (9, 0, 2)),
    (2_300_000, 16_000, 1, (5, 5, 5), (9, 0, 6)),
    (4_312_500, 30_000, 7, (6, 5, 7), (5, 5, 8)),
    (2_841_937, 19_770, 7, (6, 5, 7), (5, 5, 8)),
])
def test_msd_form_in_the_bytes_of_larger_sub_buckets(n, nodes, delay, usual, wider):
    # sub-buckets of 4,096 to 5,120 records on average, of half as many usually
    block = 1 << 18
    wl = _wl(n, nodes, delay)
    p = ng.ng_calibration_plan(n, nodes, delay)
    assert (p["b1"], p["b2"], p["b3"]) == usual
    need, least = (_msd_bytes(n, nodes, delay, block, digits=d) for d in (usual, wider))
    assert least < need
    ample = _Built(wl, "msd", block)
    tight = _Built(wl, "msd", block, ample.before + least)
    assert ample.peak - ample.before > least and tight.peak - tight.before <= least
    lsd = _Built(wl, "lsd", block)
    ample.same(lsd)
    tight.same(lsd)


def test_msd_lists_that_the_counts_cannot_hold():
    # one range: fewer of the first scatter's counts than list words
    wl = _wl(3_000_000, 100, 3)
    _Built(wl, "msd", 1 << 18, ranges=1).same(_Built(wl, "lsd", 1 << 18))


def test_default_form_goes_on_without_room_for_msd():
    # 17-bit keys: 16 bytes of scratch per connection for the MSD form, 12
    # (two passes) for the LSD form
    n, nodes, delay, block = (1 << 24) + 5, 4096, 31, 1 << 22
    wl = _wl(n, nodes, delay)
    ample = _Built(wl, "radix", block)
    assert "msd_tiles_c" in ample.kernels and "downsweep" not in ample.kernels
    blocks = -(-n // block) * 14 * block
    between = _Built(wl, "radix", block, ample.before + blocks + 14 * n)
    assert "downsweep" in between.kernels and "msd_tiles_c" not in between.kernels
    between.same(ample)
    with pytest.raises(ng.NGError) as e:  # the form asked for by name is not replaced
        _Built(wl, "msd", block, ample.before + blocks + 14 * n)
    assert e.value.status == ng.NG_ERR_OOM
    with pytest.raises(ng.NGError) as e:  # no room for either
        _Built(wl, "radix", block, ample.before + blocks + 11 * n)
    assert e.value.status == ng.NG_ERR_OOM


# The LSD form's small tiles bring more digit counts than its large ones, which
# it goes back to where the arena or the fixed scratch has no room for them.
def _lsd_bytes(n, nodes, delay, block, small, ranges=1024, radix_bits=9):
    sbits, dbits = max(nodes - 1, 0).bit_length(), delay.bit_length()
    passes = -(-(sbits + dbits) // radix_bits)
    digit = -(-(sbits + dbits) // passes)
    tile, most, gi_tile = (2048, 64 * ranges, 2048) if small else (10240, ranges, 8192)
    tiles = -(-n // tile)
    per = max(1, -(-tiles // most))
    counts = (1 << digit) * -(-tiles // per)
    gcap = min(n, nodes * delay) + 1
    gi = -(-n // gi_tile)
    sizes = [4 * n, 8 * n] * min(passes - 1, 2) + [4 * gcap, 4 * (-(-n // 32) + 1), 4 * counts,
                                                   4 * (max(-(-counts // 4096), -(-gi // 4096)) + 1), 4 * (gi + 1)]
    index = [4 * (nodes + 1), 4 * gcap]
    return sum(map(_up, sizes)), sum(map(_up, index)) + -(-n // block) * 14 * block


def test_lsd_large_tiles_where_small_ones_have_no_room():
    n, nodes, delay, block = 2_000_003, 30_000, 31, 1 << 18
    wl = _wl(n, nodes, delay)
    ample = _Built(wl, "lsd", block)
    small, large = (sum(_lsd_bytes(n, nodes, delay, block, s)) for s in (True, False))
    assert ample.peak - ample.before == small and large < small
    tight = _Built(wl, "lsd", block, ample.before + large)
    assert tight.peak - tight.before <= large
    tight.same(ample)
    with pytest.raises(ng.NGError) as e:
        _Built(wl, "lsd", block, ample.before + large - (1 << 16))
    assert e.value.status == ng.NG_ERR_OOM


def test_fixed_scratch_large_tiles_where_small_ones_have_no_room():
    nodes, delay, block = 1 << 22, 31, 1 << 18  # 27-bit keys: three passes, 512 digit values
    region = ng.ng_noalloc_scratch_bytes()
    n = next(n for n in range(2_400_000, 2_000_000, -1000)
             if _lsd_bytes(n, nodes, delay, block, False)[0] <= region)
    assert _lsd_bytes(n, nodes, delay, block, True)[0] > region
    wl = _wl(n, nodes, delay)
    fixed = _Built(wl, "lsd", block, calibrate=ng.ng_calibrate_noalloc)
    fixed.same(_Built(wl, "lsd", block))


def _copass_bytes(n, nodes, delay, block, radix_bits=9, ranges=1024):
    """Scratch and index of the in-place block sort: an auxiliary block and one
    or two sort buffers, the digit counts of one block's large tiles, the
    partition's words and copy lists, and the group index's arrays."""
    sbits, dbits = max(nodes - 1, 0).bit_length(), delay.bit_length()
    passes = -(-(sbits + dbits) // radix_bits)
    blocks, a = -(-n // block), min(n, block)
    counts = (1 << -(-(sbits + dbits) // passes)) * min(ranges, -(-a // 10240))
    gcap, gi = min(n, nodes * delay) + 1, -(-n // 8192)
    sizes = [4 * a, 8 * a] * (3 if passes >= 3 else 2)
    sizes += [4 * counts, 4 * (max(-(-counts // 4096), -(-gi // 4096)) + 1), 4 * (7 * blocks + 4), 16 * (5 * blocks + 8),
              4 * (gi + 1), 4 * gcap, 4 * (-(-n // 32) + 1), 4 * (nodes + 1), 4 * gcap]
    return sum(map(_up, sizes))


@pytest.mark.parametrize("n,nodes,delay,block", [
    (6_000_000, 50, 3, 1 << 16),             # 8-bit keys: more tiles of the group index than counts
    (800_000, 9_000, 31, 1 << 16),
    (3 * (1 << 20) + 77, 2_000, 20, 1 << 20),  # no room in the index's arrays for wider digits or more ranges
])
def test_copass_in_its_bytes(n, nodes, delay, block):
    wl = _wl(n, nodes, delay)
    need = _copass_bytes(n, nodes, delay, block)
    ample = _Built(wl, "copass", block)
    assert "copass_partition" in ample.kernels
    assert ample.peak - ample.before <= need
    tight = _Built(wl, "copass", block, ample.before + need)
    lsd = _Built(wl, "lsd", block)
    ample.same(lsd)
    tight.same(lsd)


@pytest.mark.parametrize("ns,nt", [(1500, 2000), (60_000, 50)])
def test_pairwise_leaves_no_hole_in_the_arena(ns, nt):
    # the counts and decisions of the call are gone before the calibration,
    # which fits in just its bytes above the call's blocks
    nodes, delay, block, p = 60_000, 30, 1 << 16, 0.05
    syn = ng.syn_spec(("normal", 0.5, 0.05), ("uniform_int", 1, delay))

    def build(arena):
        with Network(5, 0.1, block, arena) as net:
            net.set_calibration("lsd")
            net.create(nodes)
            _, _, n = ng.ng_connect(net.ctx, ng.ng_range(0, ns), ng.ng_range(0, nt),
                                    ng.conn_spec("pairwise_bernoulli", 0, p=p), syn)
            before = net.memory_stats()[0]
            net.calibrate()
            return n, before, net.fetch(), net.group_index()

    n, before, out, index = build(64 << 20)
    tight = build(before + sum(_lsd_bytes(n, nodes, delay, block, False)))
    assert tight[0] == n
    for k in out:
        assert np.array_equal(out[k].view(np.uint8), tight[2][k].view(np.uint8)), k
    assert np.array_equal(index[0], tight[3][0]) and np.array_equal(index[1], tight[3][1])
