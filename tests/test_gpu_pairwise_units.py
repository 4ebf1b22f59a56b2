"""pairwise_bernoulli at the edges of its units of 16,384 pairs and of the 64
pairs a thread takes, against the oracle: pair counts just below, at and just
above both, units that hold many short rows, parts of two rows or a part of
one, self-pairs left out wherever a row's falls, and the form that evaluates
the decisions again because the arena has no room to keep them."""
from types import SimpleNamespace

import numpy as np
import pytest

import oracle
from parity import check_calibrated, check_creation_order

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2306_09855_amd.network import Network  # noqa: E402

N_NODES = 50_000


def _check(calls, arena=512 << 20, seed=91):
    ns = [oracle.count_pairwise(seed, cid, c) for cid, c in enumerate(calls)]
    for c, n in zip(calls, ns):
        c.n_syn = (lambda n: lambda: n)(n)
    ref = oracle.build_network(seed, 0.1, N_NODES, calls)
    with Network(seed, 0.1, 1 << 16, arena) as net:
        net.create(N_NODES)
        assert [net.connect(c)[2] for c in calls] == ns
        check_creation_order(net.fetch(), ref, calls)
        net.calibrate()
        check_calibrated(net.fetch(), *net.group_index(), ref, calls)


def _call(ns, nt, p, first_src=0, first_tgt=0, autapses=1):
    return SimpleNamespace(rule="pairwise_bernoulli", src=(first_src, ns), tgt=(first_tgt, nt), k_or_n=0,
                           weight=("normal", 0.5, 0.05), delay=("uniform_int", 1, 25), allow_autapses=autapses, p=p)


@pytest.mark.parametrize("ns,nt", [(1, 63), (8, 8), (13, 5), (1, 16_383), (128, 128), (5, 3_277), (16_385, 1),
                                   (40_000, 3), (3, 20_000), (2, 16_384)])
def test_unit_edges(ns, nt):
    _check([_call(ns, nt, 0.3), _call(ns, nt, 0.02, 7, 11)])


@pytest.mark.parametrize("ns,nt,s0,t0", [(300, 200, 0, 100), (200, 70, 30, 0), (1_000, 3, 10, 500), (40, 20_000, 100, 0)])
def test_self_pairs_left_out(ns, nt, s0, t0):
    _check([_call(ns, nt, 1.0, s0, t0, autapses=0), _call(ns, nt, 0.4, s0, t0, autapses=0)])


def test_decisions_evaluated_again_without_room():
    # 4e8 pairs, 1 in 1e5: 50 MB of decisions do not fit an arena that holds the connections
    call = _call(20_000, 20_000, 1e-5)
    with Network(5, 0.1, 1 << 16, 32 << 20) as small, Network(5, 0.1, 1 << 16, 256 << 20) as large:
        outs = []
        for net in (small, large):
            net.create(N_NODES)
            net.connect(call)
            outs.append(net.fetch())
    for k in ("src", "tgt", "delay"):
        assert np.array_equal(outs[0][k], outs[1][k]), k
    assert np.array_equal(outs[0]["w"].view(np.uint32), outs[1]["w"].view(np.uint32))
    assert outs[0]["src"].size > 3_000
