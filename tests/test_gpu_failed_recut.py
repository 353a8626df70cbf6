"""A re-cut of the schedule whose device memory cannot be had: RS_ERR_NOMEM,
and the graph keeps its cut-offs, its schedule and its results (the allocation
is made to fail at every buffer of the new schedule in turn)."""
import os

import numpy as np
import pytest

from rsgen import lfr, pack_batch
from tests.parity import rel_close

pytestmark = pytest.mark.gpu

SMALL = {"row_entries": 256, "row_vertices": 64, "score_pairs": 64, "score_vertices": 64, "hub_list": 128}


def _results(rs, h, batch):
    out = [rs.rs_read_scores(h), *rs.rs_read_vertex_counts(h).values()]
    return out + list(rs.rs_topk_batch(h, 9) if batch else rs.rs_topk(h, 9))


@pytest.mark.parametrize("batch", [False, True])
def test_failed_recut_keeps_the_schedule(batch):
    import paper_2508_01485_amd as rs
    graphs = [lfr(n, 12.0, 700, 0.4, seed=n, cmin=10, cmax=200) for n in (1500, 900)]
    if batch:
        h = rs.rs_load_batch(*pack_batch(graphs))
    else:
        h = rs.rs_load_graph(graphs[0].off, graphs[0].col, graphs[0].labels)
    try:
        rs.rs_score(h)
        first, cut = _results(rs, h, batch), rs.rs_get_tiling(h)
        asked = 1000  # buffers asked for by the handle so far, once one has failed
        os.environ["RS_FAULT_ALLOC"] = str(asked)
        with pytest.raises(rs.RSError) as err:
            for _ in range(asked):
                rs.rs_set_tiling(h, cut)
        assert err.value.status == rs.RS_ERR_NOMEM
        rs.rs_score(h)
        failed = 0
        for i in range(1, 64):
            os.environ["RS_FAULT_ALLOC"] = str(asked + i)
            try:
                rs.rs_set_tiling(h, SMALL)
                break
            except rs.RSError as e:
                assert e.status == rs.RS_ERR_NOMEM
            asked, failed = asked + i, failed + 1
            assert rs.rs_get_tiling(h) == cut
            for a, b in zip(first, _results(rs, h, batch)):  # still scored
                assert a.tobytes() == b.tobytes()
            rs.rs_score(h)
            for a, b in zip(first, _results(rs, h, batch)):
                assert a.tobytes() == b.tobytes()
        print(f"[failed re-cut] {failed} buffers failed in turn", flush=True)
        assert failed >= 19 and rs.rs_get_tiling(h) == SMALL
        rs.rs_score(h)
        for a, b in zip(first[1:6], _results(rs, h, batch)[1:6]):
            assert np.array_equal(a, b)
        rel_close(rs.rs_read_scores(h), first[0], 1e-12)
    finally:
        os.environ.pop("RS_FAULT_ALLOC", None)
        h.free()


def test_failed_autotune_keeps_the_schedule():
    import paper_2508_01485_amd as rs
    g = lfr(1500, 12.0, 700, 0.4, seed=3, cmin=10, cmax=200)
    h = rs.rs_load_graph(g.off, g.col, g.labels)
    try:
        rs.rs_score(h)
        first, cut = _results(rs, h, False), rs.rs_get_tiling(h)
        os.environ["RS_FAULT_ALLOC"] = "1000"
        with pytest.raises(rs.RSError) as err:  # fails at some candidate after the first
            rs.rs_autotune(h, [SMALL] * 200, 1)
        assert err.value.status == rs.RS_ERR_NOMEM
        assert rs.rs_get_tiling(h) == cut
        for a, b in zip(first, _results(rs, h, False)):
            assert a.tobytes() == b.tobytes()
    finally:
        os.environ.pop("RS_FAULT_ALLOC", None)
        h.free()
