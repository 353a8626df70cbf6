"""Loads that leave the usual path: the host's build when the scratch of the
device's does not fit, and a load on a per-thread stream (the columns are
copied by another thread, whose per-thread stream is its own)."""
import os

import numpy as np
import pytest

from rsgen import lfr, pack_batch

pytestmark = pytest.mark.gpu

PER_THREAD_STREAM = 2  # hipStreamPerThread


def _results(rs, h, batch=False):
    rs.rs_score(h)
    out = [rs.rs_read_scores(h), *rs.rs_read_vertex_counts(h).values(), *rs.rs_read_rows(h), *rs.rs_read_gprime(h)]
    return out + list(rs.rs_topk_batch(h, 20) if batch else rs.rs_topk(h, 50))


def _same(a, b):
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert np.asarray(x).tobytes() == np.asarray(y).tobytes()


@pytest.mark.parametrize("flags", [0, 1])  # 1: 64-bit offsets
def test_host_build_when_the_scratch_does_not_fit(flags, monkeypatch):
    import paper_2508_01485_amd as rs
    g = lfr(7000, 14.0, 900, 0.3, seed=4, cmin=10, cmax=400)
    assert g.nnz >= 1 << 13
    off32 = g.off.astype(np.int32)
    ref = rs.rs_load_graph(g.off, g.col, g.labels, flags=flags)
    try:
        want = _results(rs, ref)
        v = np.arange(5) * 7
        res = rs.rs_apply_removals(ref, vertices=v)
        after = rs.rs_read_scores(ref)
    finally:
        ref.free()
    monkeypatch.setenv("RS_FAULT_ALLOC", "load_scratch")
    for off in (g.off, off32):
        h = rs.rs_load_graph(off, g.col, g.labels, flags=flags)
        try:
            _same(want, _results(rs, h))
            assert rs.rs_apply_removals(h, vertices=v) == res
            _same([after], [rs.rs_read_scores(h)])
        finally:
            h.free()
    col = g.col.copy()
    col[0] = g.n  # still refused, with its own status
    with pytest.raises(rs.RSError) as err:
        rs.rs_load_graph(g.off, col, g.labels, flags=flags)
    assert err.value.status == rs.RS_ERR_RANGE


def test_host_build_of_a_batch(monkeypatch):
    import paper_2508_01485_amd as rs
    packed = pack_batch([lfr(n, 12.0, 200, 0.3, seed=n, cmin=10, cmax=200) for n in (900, 2000, 150)])
    got = []
    for scratch in (True, False):
        if not scratch:
            monkeypatch.setenv("RS_FAULT_ALLOC", "load_scratch")
        h = rs.rs_load_batch(*packed)
        try:
            got.append(_results(rs, h, batch=True))
        finally:
            h.free()
    _same(*got)


@pytest.mark.parametrize("n", [300, 7000])  # built on the host, on the device
def test_per_thread_stream(n):
    import paper_2508_01485_amd as rs
    g = lfr(n, 10.0, 120, 0.3, seed=9, cmin=10, cmax=100)
    got = []
    for stream in (None, PER_THREAD_STREAM):
        h = rs.rs_load_graph(g.off, g.col, g.labels, stream=stream)
        try:
            got.append(_results(rs, h))
        finally:
            h.free()
    _same(*got)
