"""Top-k where one score class holds more vertices than are ranked pairwise
(16,384): the class is refined digit by digit down to the ids.  Equal scores
that are zero and not, k inside, at the edges of and beyond the class; the
order is descending score, then ascending id."""
import numpy as np
import pytest

from rsgen import from_edges

pytestmark = pytest.mark.gpu


def cliques(count, lone, seed):
    """Equal 4-cliques over four communities (every score the same), `lone`
    isolated vertices (score zero), and a few stars that score otherwise;
    the ids at random."""
    rng = np.random.default_rng(seed)
    base = 4 * np.arange(count)[:, None]
    pairs = np.array([(i, j) for i in range(4) for j in range(i + 1, 4)])
    e = (base[:, :, None] + pairs[None]).reshape(-1, 2)
    lab = np.tile(np.arange(4), count)
    n = 4 * count
    star = [(n, n + 1 + i) for i in range(9)] + [(n + 1, n + 2), (n + 3, n + 4)]
    lab = np.concatenate([lab, [4, 0, 1, 2, 3, 0, 1, 2, 3, 4], rng.integers(0, 5, lone)])
    e = np.concatenate([e, star])
    n = lab.size
    perm = rng.permutation(n)
    out = np.empty(n, np.int64)
    out[perm] = lab
    return from_edges(n, perm[e], out)


@pytest.mark.parametrize("count,lone", [(0, 16_400), (4097, 10), (5000, 70_000), (40_000, 3)])
def test_equal_scores(count, lone):
    import paper_2508_01485_amd as rs
    g = cliques(count, lone, 11)
    h = rs.rs_load_graph(g.off, g.col, g.labels)
    try:
        rs.rs_score(h)
        R = rs.rs_read_scores(h)
        order = np.lexsort((np.arange(g.n), -R))
        scored = int((R > 0).sum())
        for k in sorted({1, 9, 57, max(scored - 1, 1), max(scored, 1), scored + 1, scored + 5000, g.n // 2, g.n - 1, g.n}):
            if k > g.n:
                continue
            print(f"[equal scores] n={g.n} scored={scored} k={k}", flush=True)
            for _ in range(2):
                ids, sc = rs.rs_topk(h, k)
                assert np.array_equal(ids, order[:k])
                assert sc.tobytes() == R[order[:k]].tobytes()
    finally:
        h.free()
