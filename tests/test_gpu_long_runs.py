"""Long neighbour-community runs: full passes take the type-II values by slot
(workgroup tiles of 2,048 slots, a window of 4,096), incremental ones walk the
runs; both against the oracle and against each other, bit for bit.  Lengths
sit at the edges of the tile and of the window, beyond the window, and at the
row kernels' run counts."""
import numpy as np
import pytest

import oracle
from rsgen import from_edges
from tests.parity import compare, gpu_run

pytestmark = pytest.mark.gpu


def hub_runs(lengths, seed):
    """Hub i (a community of its own with two members) is joined to the first
    lengths[i][c] members of each large community c; the members have a few
    random edges inside and across communities."""
    rng = np.random.default_rng(seed)
    k = max(len(x) for x in lengths)
    size = max(max(x) for x in lengths) + 40
    first = np.arange(k) * size
    edges = []
    for c in range(k):
        m = first[c] + np.arange(size)
        edges.append(np.stack([m, first[c] + rng.integers(0, size, size)], 1))
        edges.append(np.stack([m, rng.integers(0, k * size, size)], 1))
    labels = np.repeat(np.arange(k), size).tolist()
    n = k * size
    for i, x in enumerate(lengths):
        edges.append(np.array([[n, n + 1]]))
        for c, f in enumerate(x):
            edges.append(np.stack([np.full(f, n), first[c] + np.arange(f)], 1))
        labels += [100 + i] * 2
        n += 2
    e = np.concatenate(edges)
    perm = rng.permutation(n)
    lab = np.empty(n, np.int64)
    lab[perm] = labels
    e = e[e[:, 0] != e[:, 1]]
    return from_edges(n, perm[e], lab)


CASES = {
    "short": [(2, 1, 3), (8, 9, 1), (7, 16, 17)],
    "tile_edges": [(1023, 1024, 1025), (2047, 2048, 2049), (600, 1448, 3)],
    "window_edges": [(3071, 1, 1024), (4095, 2, 4097), (1, 1, 1)],
    "beyond_window": [(6000, 5000, 1), (3, 4500, 2)],
    "many_runs": [tuple(1 + (j % 3) for j in range(m)) for m in (19, 20, 21, 63, 64, 65, 130)],
}


@pytest.mark.parametrize("name", CASES)
def test_long_runs(name):
    import paper_2508_01485_amd as rs
    g = hub_runs(CASES[name], 5)
    print(f"[long runs] {name}: n={g.n} nnz={g.nnz}", flush=True)
    gpu = gpu_run(g, 50)
    compare(g, gpu, oracle.score(g, rows=True), 50)
    h = rs.rs_load_graph(g.off, g.col, g.labels)
    try:
        rs.rs_score(h)
        u, v = g.edges()
        rng = np.random.default_rng(7)
        for _ in range(2):
            pick = rng.choice(u.size, 5, replace=False)
            rs.rs_apply_removals(h, edges=np.stack([u[pick], v[pick]], 1))
            inc = rs.rs_read_scores(h), rs.rs_read_vertex_counts(h)
            rs.rs_score(h)
            full = rs.rs_read_scores(h), rs.rs_read_vertex_counts(h)
            assert inc[0].tobytes() == full[0].tobytes()
            for key in inc[1]:
                assert inc[1][key].tobytes() == full[1][key].tobytes(), key
    finally:
        h.free()
