"""Graphs built on the device at load (from 2^13 entries on): rows at the edges
of the row kernels (64 and 65 entries, 1,024 and 1,025, several ranges of 2^20
ids), every input form against the oracle and against each other, and graphs
that are refused, with the status that small ones get."""
import numpy as np
import pytest

import oracle
from rsgen import from_edges
from tests.parity import compare, gpu_run

pytestmark = pytest.mark.gpu


def star_graph(n, rows, extra, seed, sparse_labels=False):
    """Vertex ids at random; the i-th hub gets about rows[i] neighbours on top
    of `extra` random edges, and communities come in all sizes."""
    rng = np.random.default_rng(seed)
    perm = rng.permutation(n)
    edges = [np.stack([rng.integers(len(rows), n, extra), rng.integers(len(rows), n, extra)], 1)]
    for i, d in enumerate(rows):
        edges.append(np.stack([np.full(d, i), len(rows) + rng.choice(n - len(rows), d, replace=False)], 1))
    e = perm[np.concatenate(edges)]
    e = e[e[:, 0] != e[:, 1]]
    lab = np.minimum(rng.geometric(0.05, n), 60)
    lab = lab * 30_000_001 if sparse_labels else lab * 3
    return from_edges(n, e, lab)


GRAPHS = {
    "rows": dict(n=9000, rows=(1, 63, 64, 65, 127, 128, 129, 1023, 1024, 1025, 2047, 5000), extra=40_000, seed=1),
    "sparse_labels": dict(n=8191, rows=(64, 1024, 8000), extra=30_000, seed=2, sparse_labels=True),
    "id_ranges": dict(n=(1 << 20) + 77, rows=(1024, 1025, 30_000), extra=200_000, seed=3),
    "most_in_hubs": dict(n=1300, rows=(1200,) * 40, extra=4000, seed=4),
}


@pytest.mark.parametrize("name", GRAPHS)
def test_device_load(name):
    import torch

    import paper_2508_01485_amd as rs
    g = star_graph(**GRAPHS[name])
    assert g.nnz >= 1 << 13
    print(f"[device load] {name}: n={g.n} nnz={g.nnz}", flush=True)
    first = gpu_run(g, 50)
    compare(g, first, oracle.score(g, rows=True), 50)
    off32 = g.off.astype(np.int32)
    device = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (g.off, g.col, g.labels)]
    torch.cuda.synchronize()
    for args, flags in (((off32, g.col, g.labels), 0), ((g.off, g.col, g.labels), rs.RS_LOAD_WIDE_OFFSETS),
                        (device, 0), ((device[0].int(), device[1], device[2]), rs.RS_LOAD_WIDE_OFFSETS)):
        h = rs.rs_load_graph(*args, flags=flags)
        try:
            rs.rs_score(h)
            assert rs.rs_read_scores(h).tobytes() == first["R"].tobytes()
            for key, want in rs.rs_read_vertex_counts(h).items():
                assert want.tobytes() == first[key].tobytes(), key
            for a, b in zip(rs.rs_read_gprime(h), first["gprime"]):
                assert np.asarray(a).tobytes() == np.asarray(b).tobytes()
        finally:
            h.free()


@pytest.mark.parametrize("name", ["rows", "most_in_hubs"])
def test_device_load_refuses(name):
    """One entry, offset or label changed, in a short, a middle and a long row."""
    import paper_2508_01485_amd as rs
    g = star_graph(**GRAPHS[name])
    deg = np.diff(g.off)
    order = np.argsort(deg, kind="stable")
    rows = {int(order[np.searchsorted(deg[order], lo)]) for lo in (3, 65, 1025) if deg.max() >= lo}

    def refused(off, col, lab, status):
        with pytest.raises(rs.RSError) as err:
            rs.rs_load_graph(off, col, lab)
        assert err.value.status == status

    for v in sorted(rows):
        b, e = int(g.off[v]), int(g.off[v + 1])
        print(f"[device load] refused: row of {e - b}", flush=True)
        for at, value, status in ((b, v, rs.RS_ERR_GRAPH),  # self-loop (or out of order)
                                  (b + 1, int(g.col[b]), rs.RS_ERR_GRAPH),  # a duplicate
                                  (e - 1, g.n, rs.RS_ERR_RANGE), (b, -1, rs.RS_ERR_RANGE)):
            col = g.col.copy()
            col[at] = value
            refused(g.off, col, g.labels, status)
        col = g.col.copy()  # out of order
        col[b], col[b + 1] = g.col[b + 1], g.col[b]
        refused(g.off, col, g.labels, rs.RS_ERR_GRAPH)
        # another neighbour in a gap of the row: asymmetric, otherwise sound
        gap = np.flatnonzero(np.diff(g.col[b:e]) > 2)
        free = [x for x in (int(g.col[b + i]) + 1 for i in gap) if x != v]
        if free:
            i = int(np.searchsorted(g.col[b:e], free[0])) - 1
            col = g.col.copy()
            col[b + i] = free[0]
            refused(g.off, col, g.labels, rs.RS_ERR_GRAPH)
    off = g.off.copy()
    off[5] = off[7] + 1
    refused(off, g.col, g.labels, rs.RS_ERR_GRAPH)
    off = g.off.copy()
    off[-1] -= 1  # the offsets end before the columns do
    refused(off, g.col, g.labels, rs.RS_ERR_GRAPH)
    lab = g.labels.copy()
    lab[11] = -2
    refused(g.off, g.col, lab, rs.RS_ERR_GRAPH)
