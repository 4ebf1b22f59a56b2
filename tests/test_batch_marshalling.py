"""ng_connect_batch's marshalling, without a device: whatever the lengths of the
lists, the C call gets four arrays of as many structures as it is told."""
import ctypes

import pytest

from paper_2306_09855_amd import ng


class _Recorder:
    def ng_connect_batch(self, ctx, n, srcs, tgts, conns, syns, first):
        self.n, self.arrays = n, (srcs, tgts, conns, syns)
        return ng.NG_OK


@pytest.fixture
def call(monkeypatch):
    rec = _Recorder()
    monkeypatch.setattr(ng, "lib", lambda: rec)

    def run(*lists):
        ng.ng_connect_batch(None, *lists)
        return rec

    return run


def _lists(n):
    return ([ng.ng_range(i, 1) for i in range(n)], [ng.ng_range(100 + i, 2) for i in range(n)],
            [ng.conn_spec("fixed_indegree", 3 + i) for i in range(n)],
            [ng.syn_spec(("const", 1.0 + i), ("const", 1.0)) for i in range(n)])


@pytest.mark.parametrize("n", [0, 1, 5])
def test_equal_lists_arrive_as_they_are(call, n):
    lists = _lists(n)
    rec = call(*lists)
    assert rec.n == n
    for arr, items in zip(rec.arrays, lists):
        assert len(arr) == n and bytes(arr) == b"".join(bytes(x) for x in items)


@pytest.mark.parametrize("which", [1, 2, 3])
def test_a_shorter_list_is_filled_with_zeros(call, which):
    lists = list(_lists(5))
    lists[which] = lists[which][:2]
    rec = call(*lists)
    arr, items = rec.arrays[which], lists[which]
    size = ctypes.sizeof(type(items[0]))
    assert rec.n == 5 and len(arr) == 5
    assert bytes(arr) == b"".join(bytes(x) for x in items) + bytes(3 * size)


@pytest.mark.parametrize("which", [1, 2, 3])
def test_a_longer_list_is_refused(call, which):
    lists = list(_lists(5))
    lists[which] = lists[which] + lists[which][:1]
    with pytest.raises(IndexError):
        call(*lists)


def test_other_sequences(call):
    srcs, tgts, conns, syns = _lists(4)
    rec = call(srcs, iter(tgts), tuple(conns), [s for s in syns])
    for arr, items in zip(rec.arrays, (srcs, tgts, conns, syns)):
        assert len(arr) == 4 and bytes(arr) == b"".join(bytes(x) for x in items)
