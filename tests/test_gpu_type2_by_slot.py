"""Which graphs take the type-II values by slot in a full pass: those whose
pairs would walk their runs for a quarter of the slots or more (a slot's walk:
its distance to the first of its run).  The rule is evaluated here from the
graph, so that the graphs of the long-run tests are known to take the path
that they are meant for, and one with many medium runs takes it too."""
import numpy as np
import pytest

import oracle
from tests.parity import compare, gpu_run
from tests.test_gpu_long_runs import CASES, hub_runs

pytestmark = pytest.mark.gpu

MEDIUM = [tuple(4 + (j % 9) for j in range(m)) for m in (19, 20, 21, 63, 64, 65, 130)]


def by_slot(g):
    src = np.repeat(np.arange(g.n, dtype=np.int64), np.diff(g.off))
    lab = g.labels[g.col]
    foreign = g.labels[src] != lab
    run = np.unique(src[foreign] * (int(g.labels.max()) + 1) + lab[foreign], return_counts=True)[1]
    return 4 * int((run * (run - 1) // 2).sum()) >= int(run.sum())


def test_long_run_graphs_take_the_values_by_slot():
    assert {name: by_slot(hub_runs(c, 5)) for name, c in CASES.items()} == {
        "short": True, "tile_edges": True, "window_edges": True, "beyond_window": True, "many_runs": False}
    assert by_slot(hub_runs(MEDIUM, 5))


def test_many_medium_runs():
    import paper_2508_01485_amd as rs
    g = hub_runs(MEDIUM, 5)
    compare(g, gpu_run(g, 50), oracle.score(g, rows=True), 50)
    h = rs.rs_load_graph(g.off, g.col, g.labels)
    try:
        rs.rs_score(h)
        u, v = g.edges()
        pick = np.random.default_rng(3).choice(u.size, 9, replace=False)
        rs.rs_apply_removals(h, edges=np.stack([u[pick], v[pick]], 1))  # walks the runs
        inc = rs.rs_read_scores(h), rs.rs_read_vertex_counts(h)
        rs.rs_score(h)  # by slot
        full = rs.rs_read_scores(h), rs.rs_read_vertex_counts(h)
    finally:
        h.free()
    assert inc[0].tobytes() == full[0].tobytes()
    for key in inc[1]:
        assert inc[1][key].tobytes() == full[1][key].tobytes(), key
