"""The workloads this repository is timed on: scoring passes over resident
graphs, batches of graphs, removal requests, the request server, the
reachable-community query and a one-shot run from host arrays.

Graphs follow the recipes of ``rsgen`` (LFR-style and stochastic block
graphs), drawn here with torch on the device so that graphs of tens of
millions of entries take well under a second.  ``listed`` names the cases,
``draw`` gives another of the same ranges, ``prepare`` makes a case's inputs
and handles, ``run`` is one pass as a program calls it, ``work`` counts the
bytes and operations of a pass and ``exact`` computes the scores in plain
torch, fp64, from the definitions.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2508_01485_amd as rs

# A case's fields
#   kind      "score"   rs_score + rs_topk on a resident graph
#             "readers" rs_score + every per-vertex result read back
#             "batch"   rs_score + rs_topk_batch over many graphs at once
#             "remove"  rs_apply_removals (edges and vertices) + rs_topk
#             "served"  removal requests through RSServer over several graphs
#             "reach"   rs_reachable_communities of some vertices
#             "oneshot" rs_load_graph from host arrays + rs_score + rs_topk + free
#   n, graphs vertices in all, number of graphs (batch and served: n is the
#             largest graph's, sizes are log-uniform from nmin)
#   mean, maxdeg, mix   mean and largest degree, share of edges that leave
#             their community (batch: the upper ends of the per-graph ranges)
#   cmin, cmax          community sizes; blocks: equal blocks instead, with
#             Poisson degrees
#   k         top-k (reach: the number of source vertices)
#   wide      64-bit edge offsets
#   edges, vertices     removed per request (reach: edges is the percentage
#             of all edges removed beforehand)


def listed():
    return [
        # the smallest graph a user scores: the 2,000-vertex block model,
        # top-20; latency and launches
        _case("sbm_2k", "score", n=2000, mean=6.85, maxdeg=0, mix=0.277, blocks=20, k=20),
        # an ordinary graph of the size of the robustness experiments
        _case("lfr_100k", "score", n=100_000, mean=20.0, maxdeg=1000, mix=0.1, cmin=50, cmax=5000, k=25),
        # the measured one-million-vertex workload, top-1,000
        _case("lfr_1m", "score", n=1_000_000, mean=20.0, maxdeg=5000, mix=0.1, cmin=50, cmax=20_000, k=1000),
        # the largest workload's degree and mixing law (hubs of tens of
        # thousands of neighbours), top-10,000, at a size whose inputs are
        # made in seconds
        _case("lfr_3m", "score", n=3_000_000, mean=30.0, maxdeg=100_000, mix=0.15, cmin=50, cmax=20_000, k=10_000),
        # a dense social graph (the densest mean degree of the paper's
        # datasets), heavily mixed, ragged size, 64-bit offsets
        _case("dense_150k", "score", n=150_001, mean=71.0, maxdeg=9001, mix=0.3, cmin=37, cmax=3001, k=101, wide=True),
        # all results of an ordinary graph read back
        _case("readers_300k", "readers", n=300_007, mean=14.0, maxdeg=2500, mix=0.2, cmin=20, cmax=9001, k=500),
        # the batched workload: graphs of 200 to 50,000 vertices, top-20 each
        _case("batch_128", "batch", n=50_000, nmin=200, graphs=128, mean=40.0, mix=0.3, k=20),
        # many very small graphs in one pass
        _case("batch_tiny", "batch", n=1000, nmin=20, graphs=301, mean=16.0, mix=0.3, k=7),
        # removal requests on a resident graph, each followed by a top-100
        _case("remove_1m", "remove", n=1_000_000, mean=20.0, maxdeg=5000, mix=0.1, cmin=50, cmax=20_000, k=100,
              edges=200, vertices=5),
        # eight removal requests over four resident graphs through the server
        _case("served_4", "served", n=200_000, nmin=30_000, graphs=4, mean=20.0, maxdeg=2000, mix=0.1, cmin=50,
              cmax=5000, k=100, edges=50, vertices=4),
        # the reachable-community query of the robustness experiments: 25
        # spanners and 25 random vertices, after three quarters of the edges
        # have been removed
        _case("reach_100k", "reach", n=100_000, mean=20.0, maxdeg=1000, mix=0.1, cmin=50, cmax=5000, k=50, edges=75),
        # a graph scored once, from host arrays to its top-k
        _case("oneshot_200k", "oneshot", n=200_000, mean=20.0, maxdeg=2000, mix=0.1, cmin=50, cmax=5000, k=100),
    ]


def _case(name, kind, n, mean, mix, k, maxdeg=0, cmin=0, cmax=0, blocks=0, graphs=1, nmin=0, wide=False, edges=0,
          vertices=0):
    c = dict(kind=kind, n=n, nmin=nmin or n, graphs=graphs, mean=mean, maxdeg=maxdeg, mix=mix, cmin=cmin, cmax=cmax,
             blocks=blocks, k=k, wide=wide, edges=edges, vertices=vertices)
    return c if name is None else dict(name=name, **c)


def draw(rng):
    def log(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    kind = rng.choice(["score", "score", "score", "score", "readers", "batch", "batch", "remove", "served", "reach",
                       "oneshot"])
    mean = round(log(5.0, 75.0), 2)
    mix = round(rng.uniform(0.05, 0.35), 3)
    if kind == "batch":
        nmin = int(log(20, 300))
        n = int(log(2 * nmin, 50_000))
        graphs = int(log(16, max(17, min(1000, 1_200_000 / n))))
        return _case(None, kind, n=n, nmin=nmin, graphs=graphs, mean=max(9.0, min(mean, 40.0)), mix=max(mix, 0.06),
                     k=rng.randint(1, 32))
    top = {"score": 2_000_000, "readers": 600_000, "remove": 1_000_000, "served": 200_000, "reach": 400_000,
           "oneshot": 300_000}[kind]
    low = {"score": 500, "readers": 1000, "remove": 20_000, "served": 10_000, "reach": 2000, "oneshot": 1000}[kind]
    n = int(log(low, top))
    n = min(n, int(6e7 / mean)) | rng.randint(0, 1)
    maxdeg = max(int(2 * mean), int(log(max(30.0, 3 * mean), max(31.0, 3 * mean + 1, min(n / 8, 100_000)))))
    cmin = rng.randint(10, 60)
    cmax = max(4 * cmin, int(log(100, max(200, n / 16))))
    blocks = rng.randint(2, max(3, n // 60)) if n < 50_000 and kind in ("score", "oneshot") and rng.random() < 0.3 else 0
    k = int(log(1, min(10_000, n / 2)))
    if kind == "reach":
        return _case(None, kind, n=n, mean=min(mean, 30.0), maxdeg=maxdeg, mix=mix, cmin=cmin, cmax=cmax,
                     k=rng.randint(5, 200), edges=rng.randint(60, 85))
    if kind in ("remove", "served"):
        return _case(None, kind, n=n, nmin=max(1000, n // 5), graphs=rng.randint(2, 4) if kind == "served" else 1,
                     mean=min(mean, 30.0), maxdeg=maxdeg, mix=mix, cmin=cmin, cmax=cmax, k=min(k, 1000),
                     edges=rng.randint(1, max(2, min(200, n // 400))), vertices=rng.randint(0, 4))
    return _case(None, kind, n=n, mean=mean, maxdeg=maxdeg, mix=mix, cmin=cmin, cmax=cmax, blocks=blocks, k=k,
                 wide=kind == "score" and rng.random() < 0.2)


# ------------------------------------------------------------------- inputs


def _sizes(case, rng):
    """Vertices of each graph."""
    g = case["graphs"]
    if g == 1:
        return np.array([case["n"]], np.int64)
    return np.exp(rng.uniform(math.log(case["nmin"]), math.log(case["n"]), g)).round().astype(np.int64)


def _degree_floor(mean, hi, expo=2.5):
    """x0 of the density x^-expo on [x0, hi] whose mean is `mean` (arrays)."""
    lo, up = np.full(mean.shape, 0.5), np.minimum(mean, hi)
    for _ in range(60):
        x = 0.5 * (lo + up)
        got = (x ** (2 - expo) - hi ** (2 - expo)) / (x ** (1 - expo) - hi ** (1 - expo)) * (expo - 1) / (expo - 2)
        lo, up = np.where(got < mean, x, lo), np.where(got < mean, up, x)
    return 0.5 * (lo + up)


def _graphs(case, seed):
    """The case's graphs as one disjoint union on the device: (vertex starts
    [G+1] on the host, src, dst of every CSR entry ascending, labels)."""
    dev = torch.device("cuda")
    rng = np.random.default_rng([seed, 77])
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(rng.integers(1 << 40)))

    def uniform(size):
        return torch.rand(size, generator=gen, device=dev, dtype=torch.float64)

    ns = _sizes(case, rng)
    G = ns.size
    vo = np.concatenate([[0], np.cumsum(ns)])
    N = int(vo[-1])
    # per graph: mean degree, largest degree, mixing, community sizes, law
    if case["kind"] == "batch":
        mean = rng.uniform(8.0, case["mean"], G)
        mix = rng.uniform(0.05, case["mix"], G)
        hi = np.minimum(1000.0, np.maximum(ns / 4.0, 4.0))
        ncom = np.minimum(rng.integers(5, 501, G), np.maximum(ns // 10, 1))
        block = rng.random(G) < 0.5
        s_lo, s_hi = ns / ncom / 4.0, 4.0 * ns / ncom
    else:
        mean, mix = np.full(G, case["mean"]), np.full(G, case["mix"])
        hi = np.minimum(float(case["maxdeg"] or 1), ns / 2.0)
        block = np.full(G, case["blocks"] > 0)
        if case["blocks"]:
            ncom = np.full(G, case["blocks"])
            s_lo = s_hi = ns / ncom
        else:
            s_hi = np.minimum(float(case["cmax"]), np.maximum(ns / 4.0, 4.0))
            s_lo = np.minimum(float(case["cmin"]), s_hi / 2.0)
            ncom = np.maximum(2, np.round(ns / np.sqrt(s_lo * s_hi))).astype(np.int64)
    mean = np.minimum(mean, np.maximum(ns / 3.0, 1.0))
    hi = np.maximum(hi, mean + 1.0)
    # communities: sizes from s^-1.5 (or equal), as shares of the graph
    cg = np.repeat(np.arange(G), ncom)
    u = rng.random(cg.size)
    a, b = s_lo[cg] ** -0.5, s_hi[cg] ** -0.5
    share = np.where(block[cg], 1.0, (a - u * (a - b)) ** -2.0)
    tot = np.bincount(cg, share, G)
    csize = np.maximum(1, np.round(share / tot[cg] * ns[cg])).astype(np.int64)
    order = np.lexsort((-csize, cg))
    csize, cg = csize[order], cg[order]
    C = cg.size
    first = np.concatenate([[0], np.cumsum(ncom)])
    # degrees
    gv = torch.repeat_interleave(torch.arange(G, device=dev), torch.from_numpy(ns).to(dev))
    x0, hi_t = torch.from_numpy(_degree_floor(mean + 0.5, hi + 1.0)).to(dev)[gv], torch.from_numpy(hi).to(dev)[gv]
    A, B = x0 ** -1.5, (hi_t + 1.0) ** -1.5
    deg = torch.minimum(torch.floor((A - uniform(N) * (A - B)) ** (-1.0 / 1.5)), torch.floor(hi_t))
    mean_t = torch.from_numpy(mean).to(dev)[gv]
    pois = torch.poisson(mean_t, generator=gen)
    deg = torch.where(torch.from_numpy(block).to(dev)[gv], pois, deg).long()
    k_ext = torch.floor(torch.from_numpy(mix).to(dev)[gv] * deg + uniform(N)).long()
    k_in = deg - k_ext
    # each vertex joins a community larger than its internal degree, with
    # probability proportional to size (the largest one if none is)
    csum = torch.from_numpy(np.cumsum(csize).astype(np.float64)).to(dev)
    base = torch.from_numpy(np.concatenate([[0.0], np.cumsum(csize).astype(np.float64)])[first[:-1]]).to(dev)[gv]
    key = torch.from_numpy(cg.astype(np.int64) * (1 << 32) - csize).to(dev)
    f_t = torch.from_numpy(first[:-1]).to(dev)[gv]
    elig = torch.searchsorted(key, gv * (1 << 32) - k_in)
    elig = torch.where(torch.from_numpy(block).to(dev)[gv], torch.from_numpy(first[1:]).to(dev)[gv],
                       torch.maximum(elig, f_t + 1))
    com = torch.searchsorted(csum, base + uniform(N) * (csum[elig - 1] - base), right=True)
    com = torch.minimum(torch.maximum(com, f_t), elig - 1)
    over = torch.clamp(k_in - torch.clamp(torch.bincount(com, minlength=C)[com] - 1, min=0), min=0)
    k_in, k_ext = k_in - over, k_ext + over
    # pair the stubs inside each community, then across communities inside
    # each graph (same-community pairs are drawn again a few times)
    keys = []

    def pair(stubs, group, foreign):
        stubs = stubs[torch.argsort(uniform(stubs.numel()), stable=True)]
        stubs = stubs[torch.argsort(group[stubs], stable=True)]
        h = stubs.numel() // 2
        a, b = stubs[0:2 * h:2], stubs[1:2 * h:2]
        ok = (group[a] == group[b]) & (a != b)
        if foreign:
            ok &= com[a] != com[b]
        keys.append(torch.minimum(a[ok], b[ok]) * N + torch.maximum(a[ok], b[ok]))
        return torch.cat([a[~ok], b[~ok]])

    ids = torch.arange(N, device=dev)
    pair(torch.repeat_interleave(ids, k_in), com, False)
    rest = torch.repeat_interleave(ids, k_ext)
    for _ in range(3):
        if rest.numel() > 1:
            rest = pair(rest, gv, True)
    # random vertex ids inside each graph, random community labels
    pos = torch.argsort(uniform(N), stable=True)
    pos = pos[torch.argsort(gv[pos], stable=True)]
    new = torch.empty_like(pos)
    new[pos] = ids
    key = torch.unique(torch.cat(keys))
    a, b = new[key // N], new[key % N]
    both = torch.sort(torch.cat([a * N + b, b * N + a]))[0]
    perm = torch.argsort(uniform(C), stable=True)
    lab = torch.empty(N, dtype=torch.int64, device=dev)
    lab[new] = perm[com]
    return vo, both // N, both % N, lab


def _csr(n, src, dst, lab):
    off = torch.zeros(n + 1, dtype=torch.int64, device=src.device)
    torch.cumsum(torch.bincount(src, minlength=n), 0, out=off[1:])
    return off, dst.int(), lab.int()


def _host(csr):
    return tuple(t.cpu().numpy() for t in csr)


def _split(vo, src, dst, lab):
    """The union's graphs one by one, as (n, src, dst, labels)."""
    cut = torch.searchsorted(src, torch.from_numpy(vo).to(src.device)).tolist()
    return [(int(vo[i + 1] - vo[i]), src[cut[i]:cut[i + 1]] - int(vo[i]), dst[cut[i]:cut[i + 1]] - int(vo[i]),
             lab[int(vo[i]):int(vo[i + 1])]) for i in range(vo.size - 1)]


MOST_EDGES = 4_000_000


def _requests(case, n, src, dst, seed):
    """Edges and vertices to remove, in the order the requests take them."""
    rng = np.random.default_rng([seed, 78])
    up = src < dst
    a, b = src[up], dst[up]
    m = a.numel()
    pick = torch.from_numpy(rng.permutation(m)[:min(m, MOST_EDGES)]).to(a.device)
    e = torch.stack([a[pick], b[pick]], 1).int().cpu().numpy()
    return e, rng.permutation(n).astype(np.int32)


def _batch_of(case, req, i):
    """The i-th request's edges and vertices (around again at the end)."""
    e, v = req
    ne, nv = max(1, min(case["edges"], e.shape[0])), case["vertices"]
    i_e, i_v = i % max(1, e.shape[0] // ne), i % max(1, v.size // max(nv, 1))
    return e[i_e * ne:(i_e + 1) * ne], v[i_v * nv:(i_v + 1) * nv]


def prepare(case, seed):
    kind = case["kind"]
    vo, src, dst, lab = _graphs(case, seed)
    N = int(vo[-1])
    st = {"case": case}
    if kind == "batch":
        st["h"] = rs.rs_load_batch(vo, *_host(_csr(N, src, dst, lab)))
    elif kind == "served":
        st["srv"], st["req"], st["at"] = rs.rs_server_create(slots=case["graphs"]), [], 0
        for i, (n, s, d, l) in enumerate(_split(vo, src, dst, lab)):
            rs.rs_server_add_graph(st["srv"], *_host(_csr(n, s, d, l)))
            st["req"].append(_requests(case, n, s, d, seed + 1000 * (i + 1)))
        # one empty request a graph: the graphs are resident before the first pass
        for r in [rs.rs_server_submit(st["srv"], i, 1) for i in range(case["graphs"])]:
            rs.rs_server_wait(st["srv"], r)
    elif kind == "oneshot":
        st["csr"] = _host(_csr(N, src, dst, lab))
    else:
        st["h"] = rs.rs_load_graph(*_csr(N, src, dst, lab), flags=rs.RS_LOAD_WIDE_OFFSETS if case["wide"] else 0)
        if kind == "remove":
            st["req"], st["at"] = _requests(case, N, src, dst, seed), 0
            rs.rs_score(st["h"])
            rs.rs_topk(st["h"], case["k"])
        elif kind == "reach":
            e = _requests(case, N, src, dst, seed)[0]
            rs.rs_score(st["h"])
            rs.rs_apply_removals(st["h"], edges=e[:src.numel() // 2 * case["edges"] // 100])
            st["sources"] = np.random.default_rng([seed, 79]).permutation(N)[:case["k"]].astype(np.int32)
    return st


def run(state):
    case = state["case"]
    kind, k = case["kind"], case["k"]
    if kind == "score":
        rs.rs_score(state["h"])
        return dict(zip(("ids", "scores"), rs.rs_topk(state["h"], k)))
    if kind == "batch":
        rs.rs_score(state["h"])
        return dict(zip(("ids", "scores", "counts"), rs.rs_topk_batch(state["h"], k)))
    if kind == "readers":
        rs.rs_score(state["h"])
        out = rs.rs_read_vertex_counts(state["h"])
        out["R"] = rs.rs_read_scores(state["h"])
        out["ids"], out["scores"] = rs.rs_topk(state["h"], k)
        return out
    if kind == "remove":
        e, v = _batch_of(case, state["req"], state["at"])
        state["at"] += 1
        out = rs.rs_apply_removals(state["h"], edges=e, vertices=v)
        out["ids"], out["scores"] = rs.rs_topk(state["h"], k)
        return out
    if kind == "served":
        out, asked = [], []
        for _ in range(2):
            for i in range(case["graphs"]):
                e, v = _batch_of(case, state["req"][i], state["at"])
                asked.append(rs.rs_server_submit(state["srv"], i, k, edges=e, vertices=v))
            state["at"] += 1
        for r in asked:
            ids, scores, _ = rs.rs_server_wait(state["srv"], r)
            out.append({"ids": ids, "scores": scores})
        return out
    if kind == "reach":
        return rs.rs_reachable_communities(state["h"], state["sources"])
    h = rs.rs_load_graph(*state["csr"])
    rs.rs_score(h)
    ids, scores = rs.rs_topk(h, k)
    rs.rs_free_graph(h)
    return {"ids": ids, "scores": scores}


def work(case):
    """Bytes: offsets, columns and labels read once, results written once.
    Operations: a dozen for each entry (the row statistics and the foreign
    pairs' terms)."""
    n = float(case["n"])
    if case["graphs"] > 1:
        lo = max(float(case["nmin"]), 1.0)
        n = case["graphs"] * ((n - lo) / math.log(n / lo) if n > lo else n)
    nnz = n * (0.5 * (8.0 + case["mean"]) if case["kind"] == "batch" else case["mean"])
    out = 12.0 * case["k"] * (case["graphs"] if case["kind"] == "batch" else 1)
    if case["kind"] == "readers":
        out += n * (12 + 16 + 16)
    if case["kind"] == "reach":
        return {"bytes": 4 * n + 4 * nnz + 4 * n + 12 * case["k"], "flops": nnz}
    if case["kind"] in ("remove", "served"):
        # a request reads the scores for its top-k, and the changed rows and
        # those next to them (a fiftieth of the graph stands for them)
        one = 8 * n + (8 * n + 4 * nnz) / 50 + 8.0 * case["edges"] + out
        return {"bytes": one * (2 if case["kind"] == "served" else 1), "flops": 12 * nnz / 50}
    return {"bytes": 4 * n + 4 * nnz + 4 * n + out, "flops": 12 * nnz}


# -------------------------------------------------------------------- exact


def _weights(n, K, src, c_dst, lab):
    """Records (vertex, community) of the interaction matrix: sorted keys,
    counts, weights w_v(c), and each vertex's own weight; w_max's argument."""
    key, f = torch.unique(src * K + c_dst, return_counts=True)
    v, c = key // K, key % K
    f = f.double()
    d = torch.bincount(src, minlength=n).double()
    ell = torch.bincount(v, minlength=n).double()
    X = torch.zeros(n, dtype=torch.float64, device=src.device).index_add_(0, v, f * torch.log2(f))

    def weight(others, Y, X):
        ok = (others > 1) & (Y > 0)
        Ys = torch.where(ok, Y, torch.ones_like(Y))
        return torch.where(ok, others * (torch.log2(Ys) - X / Ys), torch.zeros_like(Y))

    w = weight(ell[v] - 1, d[v] - f, X[v] - f * torch.log2(f))
    own = weight(ell, d, X)  # the own community absent among the neighbours
    mine = c == lab[v]
    own[v[mine]] = w[mine]
    return key, w, own, d


def _scores(n, src, dst, lab, graph=None, n_graphs=1):
    """R of every vertex (each graph of a union by its own w_max), its border
    flag, and w_v(C(v)), in fp64 from the definitions."""
    dev = src.device
    lab = torch.unique(lab, return_inverse=True)[1]
    K = int(lab.max()) + 1 if n else 1
    key, w, own, d = _weights(n, K, src, lab[dst], lab)
    a = own.clamp(min=0).pow(1.0 / 3.0)
    graph = torch.zeros(n, dtype=torch.int64, device=dev) if graph is None else graph
    foreign = lab[src] != lab[dst]
    fu, fw = src[foreign], dst[foreign]
    border = torch.zeros(n, dtype=torch.bool, device=dev)
    border[fu] = True
    best = torch.zeros(n, dtype=torch.float64, device=dev).scatter_reduce_(0, key // K, w, "amax")
    best = torch.where(border, torch.maximum(best, own), torch.zeros_like(own))
    wmax = torch.zeros(n_graphs, dtype=torch.float64, device=dev).scatter_reduce_(0, graph, best, "amax")
    w = w.clamp(min=0)

    def w_of(v, c):
        return w[torch.searchsorted(key, v * K + c)]

    raw = torch.zeros(n, dtype=torch.float64, device=dev)
    # type II: u's foreign neighbour w and w's other neighbours in C(u)
    sums = torch.zeros(key.numel(), dtype=torch.float64, device=dev)
    at = torch.searchsorted(key, src * K + lab[dst])
    sums.index_add_(0, at, a[dst])
    rec = torch.searchsorted(key, fw * K + lab[fu])
    raw.index_add_(0, fu, w[rec].pow(2.0 / 3.0) * (sums[rec] - a[fu]).clamp(min=0))
    # type I: triangles of foreign edges, each found once by lifting every
    # edge to its higher-degree end
    fd = torch.bincount(fu, minlength=n)
    rank = fd * n + torch.arange(n, device=dev)
    up = rank[fw] > rank[fu]
    x, y = fu[up], fw[up]
    edge = fu * n + fw  # ascending: the entries are
    off = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    torch.cumsum(torch.bincount(x, minlength=n), 0, out=off[1:])
    reps = off[y + 1] - off[y]
    ends = torch.cumsum(reps, 0)
    lo = 0
    while lo < x.numel():
        done = int(ends[lo - 1]) if lo else 0
        hi = max(lo + 1, int(torch.searchsorted(ends, done + 50_000_000, right=True)))
        r = reps[lo:hi]
        i = torch.repeat_interleave(torch.arange(lo, min(hi, x.numel()), device=dev), r)
        z = y[off[y[i]] + torch.arange(i.numel(), device=dev) - (ends[i] - reps[i] - done)]
        p, q = x[i], y[i]
        want = p * n + z
        got = torch.searchsorted(edge, want).clamp(max=max(edge.numel() - 1, 0))
        hit = edge[got] == want
        t = (p[hit], q[hit], z[hit])
        for u, s, v in ((0, 1, 2), (1, 0, 2), (2, 0, 1)):
            for s2, v2 in ((s, v), (v, s)):
                U, W, V = t[u], t[s2], t[v2]
                term = (w_of(V, lab[U]) * w_of(W, lab[V]) * w_of(W, lab[U])).pow(1.0 / 3.0)
                raw.index_add_(0, U, term)
        lo = hi
    den = wmax[graph] * d * (d - 1)
    R = torch.where((den > 0) & (d >= 2), raw / torch.where(den > 0, den, torch.ones_like(den)), torch.zeros_like(raw))
    return R, border, own


def _top(R, alive, k):
    R = R[alive]
    return torch.sort(R, descending=True)[0][:min(k, R.numel())]


def _without(n, src, dst, gone_e, dead):
    keep = ~(dead[src] | dead[dst])
    if len(gone_e):
        g = torch.from_numpy(gone_e.astype(np.int64)).to(src.device)
        bad = torch.sort(torch.cat([g[:, 0] * n + g[:, 1], g[:, 1] * n + g[:, 0]]))[0]
        key = src * n + dst
        keep &= bad[torch.searchsorted(bad, key).clamp(max=bad.numel() - 1)] != key
    return src[keep], dst[keep]


def exact(case, seed):
    kind, k = case["kind"], case["k"]
    if kind == "reach":
        return None  # whole numbers
    vo, src, dst, lab = _graphs(case, seed)
    n = int(vo[-1])
    if kind == "served":
        out = [None] * (2 * case["graphs"])
        for i, (gn, s, d, l) in enumerate(_split(vo, src, dst, lab)):
            req = _requests(case, gn, s, d, seed + 1000 * (i + 1))
            dead = torch.zeros(gn, dtype=torch.bool, device=s.device)
            gone = np.zeros((0, 2), np.int32)
            for j in range(2):
                e, v = _batch_of(case, req, j)
                gone = np.concatenate([gone, e])
                dead[torch.from_numpy(v.astype(np.int64)).to(s.device)] = True
                s2, d2 = _without(gn, s, d, gone, dead)
                out[j * case["graphs"] + i] = {"ids": None, "scores": _top(_scores(gn, s2, d2, l)[0], ~dead, k)}
        return out
    alive = torch.ones(n, dtype=torch.bool, device=src.device)
    if kind == "remove":
        e, v = _batch_of(case, _requests(case, n, src, dst, seed), 0)
        alive[torch.from_numpy(v.astype(np.int64)).to(src.device)] = False
        src, dst = _without(n, src, dst, e, ~alive)
        out = dict.fromkeys(("edges_removed", "edges_ignored", "vertices_removed", "affected", "ids"))
        return dict(out, scores=_top(_scores(n, src, dst, lab)[0], alive, k))
    if kind == "batch":
        G = vo.size - 1
        graph = torch.repeat_interleave(torch.arange(G, device=src.device), torch.from_numpy(np.diff(vo)).to(src.device))
        R = _scores(n, src, dst, lab, graph, G)[0]
        scores = torch.zeros(G, k, dtype=torch.float64, device=src.device)
        for i in range(G):
            t = torch.sort(R[int(vo[i]):int(vo[i + 1])], descending=True)[0][:k]
            scores[i, :t.numel()] = t
        return {"ids": None, "scores": scores, "counts": None}
    R, border, own = _scores(n, src, dst, lab)
    top = {"ids": None, "scores": _top(R, alive, k)}
    if kind == "readers":
        return dict(top, border=border.int(), ell=None, dprime=None, tI=None, tII=None, w_own=own, R=R)
    return top
