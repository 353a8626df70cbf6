"""The batched top-k at the edges of its segments (1,024 vertices), with few and
many segments a graph, all-equal and mostly zero scores (ids decide), empty
graphs and graphs smaller than k; against the lone graph's top-k."""
import numpy as np
import pytest

from rsgen import Graph, from_edges, pack_batch

pytestmark = pytest.mark.gpu


def cliques(n, every, rng):
    """Disjoint 4-cliques over four communities on every `every`-th block of
    four vertices; the other vertices are isolated (score zero)."""
    e = []
    for b in range(0, n - 3, 4 * every):
        v = b + np.arange(4)
        e += [(v[i], v[j]) for i in range(4) for j in range(i)]
    p = rng.permutation(n)
    e = p[np.array(e).reshape(-1, 2)] if e else np.zeros((0, 2), np.int64)
    lab = np.empty(n, np.int32)
    lab[p] = np.arange(n) % 4
    return from_edges(n, e, lab)


@pytest.mark.parametrize("k", [1, 2, 19, 32])
@pytest.mark.parametrize("sizes", [(1, 3, 5, 31, 32, 33, 63, 64, 65, 0, 200),
                                   (1023, 1024, 1025, 2047, 2048, 2049, 0, 1), (5000, 20000, 40000, 33)])
def test_batch_topk_edges(sizes, k):
    import paper_2508_01485_amd as rs
    rng = np.random.default_rng([k, len(sizes)])
    gs = [cliques(n, int(rng.integers(1, 6)), rng) if n else
          Graph(0, np.zeros(1, np.int64), np.zeros(0, np.int32), np.zeros(0, np.int32)) for n in sizes]
    h = rs.rs_load_batch(*pack_batch(gs))
    try:
        rs.rs_score(h)
        for _ in range(2):
            ids, sc, cnt = rs.rs_topk_batch(h, k)
            for i, g in enumerate(gs):
                c = min(k, g.n)
                assert cnt[i] == c, i
                if not c:
                    continue
                a = rs.rs_load_graph(g.off, g.col, g.labels)
                rs.rs_score(a)
                ref = rs.rs_topk(a, k)
                a.free()
                assert np.array_equal(ids[i, :c], ref[0]), i
                assert sc[i, :c].tobytes() == ref[1].tobytes(), i
                assert not ids[i, c:].any() and not sc[i, c:].any()
    finally:
        h.free()
