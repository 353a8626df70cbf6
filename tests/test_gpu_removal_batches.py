"""Removal batches around the limits of the one-launch path: ids read from
pinned memory or copied (8,192 ids), listed edges at listed vertices (two
launches) or apart from them (one), up to 16,384 edges and beyond, and rows of
many 64-entry chunks that lose all their entries.  The counts against a plain
count on the host, the scores against a full pass, bit for bit."""
import numpy as np
import pytest

from rsgen import from_edges

pytestmark = pytest.mark.gpu


def graph(n=30_000, seed=3):
    rng = np.random.default_rng(seed)
    e = rng.integers(0, n, (6 * n, 2))
    hub = np.stack([np.zeros(5000, np.int64), 1 + rng.choice(n - 1, 5000, replace=False)], 1)
    big = np.stack([np.ones(70, np.int64), 2 + rng.choice(n - 2, 70, replace=False)], 1)
    e = np.concatenate([e, hub, big])
    return from_edges(n, e[e[:, 0] != e[:, 1]], rng.integers(0, 300, n) ** 2 // 300)


def live_edges(edges, gone_e, gone_v):
    """(edges removed as listed, edges removed with vertices, edges left)"""
    key = edges[:, 0] << 32 | edges[:, 1]
    drop = np.unique(np.sort(gone_e.astype(np.int64), axis=1) @ np.array([1 << 32, 1]))
    listed = np.isin(key, drop)
    at_v = ~listed & np.isin(edges, gone_v).any(1)
    return int(listed.sum()), int(at_v.sum()), edges[~listed & ~at_v]


@pytest.mark.parametrize("m,nv,overlap", [(1, 0, False), (0, 1, False), (64, 3, True), (64, 3, False),
                                          (4093, 5, False), (4094, 4, False), (4094, 5, True), (8191, 2, False),
                                          (16_384, 40, False), (16_384, 40, True), (16_385, 40, False)])
def test_removal_batches(m, nv, overlap):
    import paper_2508_01485_amd as rs
    g = graph()
    u, v = g.edges()
    edges = np.sort(np.stack([u, v], 1).astype(np.int64), axis=1)
    rng = np.random.default_rng(m + nv)
    h = rs.rs_load_graph(g.off, g.col, g.labels)
    try:
        rs.rs_score(h)
        live = np.arange(g.n)
        for step in range(3):
            verts = rng.choice(live, nv, replace=False)
            if nv and step == 0:
                verts = np.append(verts[verts != 0][:nv - 1], 0)  # with the hub
            live = np.setdiff1d(live, verts)
            at = np.isin(edges, verts).any(1)
            if overlap:  # edges at the vertices first
                order = np.concatenate([rng.permutation(np.flatnonzero(at)), rng.permutation(np.flatnonzero(~at))])
            else:
                order = rng.permutation(np.flatnonzero(~at))
            pick = edges[order[:m]].copy()
            if m > 2:
                pick[1] = pick[0][::-1]  # a duplicate, the other way round
                pick[2] = (pick[0][0], pick[0][0])  # no edge at all
            print(f"[removal] m={m} nv={nv} overlap={overlap} step={step}", flush=True)
            res = rs.rs_apply_removals(h, edges=pick, vertices=verts)
            listed, with_v, edges = live_edges(edges, pick, verts)
            assert res["edges_removed"] == listed + with_v
            assert res["edges_ignored"] == m - listed
            assert res["vertices_removed"] == nv
            inc = rs.rs_read_scores(h), rs.rs_read_vertex_counts(h), rs.rs_topk(h, 100)
            rs.rs_score(h)
            full = rs.rs_read_scores(h), rs.rs_read_vertex_counts(h), rs.rs_topk(h, 100)
            assert inc[0].tobytes() == full[0].tobytes()
            for key in inc[1]:
                assert inc[1][key].tobytes() == full[1][key].tobytes(), key
            for a, b in zip(inc[2], full[2]):
                assert a.tobytes() == b.tobytes()
            c = rs.rs_read_counts(h)
            assert c["n_alive"] == live.size and c["nnz"] == 2 * len(edges)
    finally:
        h.free()
