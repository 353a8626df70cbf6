"""Reachable communities where the union-find and the bitmaps change path: rows
around the lane/wavefront cut (16 entries), long chains, all sources in one
component, bitmaps within and beyond the workgroup's LDS (8,192 words),
repeated sources; against the oracle's searches."""
import numpy as np
import pytest

import oracle
from rsgen import from_edges

pytestmark = pytest.mark.gpu


def chain(n, rng):
    p = rng.permutation(n)
    return np.stack([p[:-1], p[1:]], 1)


def stars(sizes, rng):
    e, at = [], 0
    for s in sizes:
        e.append(np.stack([np.full(s, at), at + 1 + np.arange(s)], 1))
        at += s + 1
    return np.concatenate(e), at


@pytest.mark.parametrize("shape,k,ns", [("chain", 5, 3), ("stars", 40, 64), ("stars", 900, 1024), ("pairs", 3, 1000),
                                        ("random", 33, 250), ("random", 2000, 200)])
def test_reach_shapes(shape, k, ns):
    import paper_2508_01485_amd as rs
    rng = np.random.default_rng([len(shape), k, ns])
    n = 3000
    if shape == "chain":
        e = chain(n, rng)
    elif shape == "stars":
        e, used = stars((1, 2, 15, 16, 17, 18, 63, 79, 80, 81, 500, 1200), rng)
        assert used <= n
    elif shape == "pairs":
        e = np.stack([np.arange(0, n, 2), np.arange(1, n, 2)], 1)
    else:
        e = rng.integers(0, n, (n, 2))
        e = e[e[:, 0] != e[:, 1]]
    perm = rng.permutation(n)
    g = from_edges(n, perm[e], rng.integers(0, k, n))
    src = rng.integers(0, n, ns)  # with repeats
    h = rs.rs_load_graph(g.off, g.col, g.labels)
    try:
        exp = oracle.reachable_communities(g, src)
        for _ in range(2):
            assert np.array_equal(rs.rs_reachable_communities(h, src), exp)
            assert np.array_equal(rs.rs_reachable_communities_static(h, src), exp)
    finally:
        h.free()
