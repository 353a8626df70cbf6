"""The server's memory budget: a graph is admitted by the sizes of its own
buffers, whatever the share of its edges between communities, and results are
those of a lone handle."""
import numpy as np
import pytest

from rsgen import from_edges, lfr
from tests.test_gpu_served import _alone, _compare, _served

pytestmark = pytest.mark.gpu


def _per_entry_guess(g):
    """A size from the vertices and entries alone, which is too much for a graph
    with few edges between communities and too little for one with most."""
    return 48 * g.nnz + 360 * g.n + (8 << 20)


def test_graph_with_few_foreign_edges_fits():
    import paper_2508_01485_amd as rs
    g = lfr(60_000, 14.0, 500, 0.05, seed=5, cmin=20, cmax=600)
    reqs = [(0, None, np.array([3])), (0, None, np.array([4, 5]))]
    budget = _per_entry_guess(g) * 2 // 3
    served, st = _served(rs, [g], reqs, 20, slots=1, budget=budget)
    _compare(_alone(rs, [g], reqs, 20), served)
    assert st["loads"] == 1 and st["evictions"] == 0 and st["peak_device_bytes"] <= budget, st
    print("[served budget] few foreign edges", budget, st, flush=True)


def test_graphs_of_foreign_edges_wait_for_room():
    """Two graphs with nearly all edges between communities, requested at once
    under a budget that holds one of them: the second waits for the first."""
    import paper_2508_01485_amd as rs
    rng = np.random.default_rng(8)
    n, m = 3000, 800_000
    graphs = [from_edges(n, rng.integers(0, n, (m, 2)), rng.integers(0, 300, n)) for _ in range(2)]
    src = [np.repeat(np.arange(n), np.diff(g.off)) for g in graphs]
    assert all((g.labels[s] != g.labels[g.col]).mean() > 0.99 for g, s in zip(graphs, src))
    reqs = [(i % 2, None, np.array([10 + i])) for i in range(6)]
    budget = 2 * max(_per_entry_guess(g) for g in graphs) + (1 << 20)
    served, st = _served(rs, graphs, reqs, 15, slots=2, budget=budget)
    _compare(_alone(rs, graphs, reqs, 15), served)
    assert st["peak_device_bytes"] <= budget and st["evictions"] > 0, st
    print("[served budget] foreign edges", budget, st, flush=True)


def test_small_graphs_stay_resident():
    """Forty graphs of 200 vertices (half a MiB of buffers each) under 96 MiB:
    none is evicted, and the budget's account is near what the device gave away."""
    import torch

    import paper_2508_01485_amd as rs
    graphs = [lfr(200, 8.0, 50, 0.25, seed=i, cmin=10, cmax=60) for i in range(40)]
    reqs = [(i % 40, None, np.array([i % 7])) for i in range(80)]
    alone = _alone(rs, graphs, reqs, 10)  # (also the process's first streams)
    srv = rs.RSServer(slots=2, hbm_budget=96 << 20)
    try:
        free = torch.cuda.mem_get_info()[0]
        gids = [srv.add_graph(g.off, g.col, g.labels) for g in graphs]
        rids = [srv.submit(gids[gi], 10, vertices=v) for gi, _, v in reqs]
        served = [srv.wait(r) for r in rids]
        taken, st = free - torch.cuda.mem_get_info()[0], srv.stats()
    finally:
        srv.free()
    _compare(alone, served)
    print("[served budget] small graphs", st, "device", taken, flush=True)
    assert st["evictions"] == 0 and st["loads"] == 40, st
    # 60 MiB; within a quarter and two chunks for sharing and the allocator's state
    assert abs(st["device_bytes"] - taken) <= taken // 4 + (4 << 20), (st, taken)
