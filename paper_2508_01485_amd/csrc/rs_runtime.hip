// rs_runtime.hip -- host side of the RS library: the C ABI of include/rs.h.
//
// rs_load_graph validates the caller's CSR (a simple undirected graph,
// Section II), renumbers it so that every community is a contiguous id range
// (labels ascending, caller ids ascending inside a community), re-sorts the
// rows and cuts the schedule of tiles and hubs, into device memory owned by the
// handle (large graphs: the rows are checked, renumbered and sorted on the
// device).  All later calls run kernels on the graph's stream (rs_kernels.hip);
// the host only marshals arguments, sizes launches and copies results.
#include <algorithm>
#include <array>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <new>
#include <thread>

#include "rs_internal.h"

namespace rs {

static thread_local std::string g_err;

rs_status fail(rs_status s, const std::string &msg) {
    g_err = msg;
    return s;
}

rs_status hip_fail(hipError_t e, const char *what) {
    g_err = std::string(what) + ": " + hipGetErrorString(e);
    return (e == hipErrorOutOfMemory) ? RS_ERR_NOMEM : RS_ERR_HIP;
}

void clear_error() { g_err.clear(); }

// ------------------------------------------------------------ host threads
template <class F>
static void parallel_for(int64_t n, int64_t grain, F &&f) {
    unsigned nt = std::thread::hardware_concurrency();
    nt = std::max(1u, std::min(nt, 16u));
    if (n <= grain || nt == 1) {
        f((int64_t)0, n);
        return;
    }
    std::atomic<int64_t> next{0};
    auto work = [&]() {
        for (;;) {
            int64_t s = next.fetch_add(grain);
            if (s >= n) break;
            f(s, std::min(n, s + grain));
        }
    };
    std::vector<std::thread> th;
    th.reserve(nt - 1);
    for (unsigned i = 1; i < nt; ++i) {
        try {
            th.emplace_back(work);
        } catch (...) {  // no more threads: those there do the rest
            break;
        }
    }
    work();
    for (auto &t : th) t.join();
}

// ------------------------------------------------------------ allocation
// Optional fault injection for tests of the error paths: RS_FAULT_ALLOC=N
// makes the N-th buffer that a handle asks for fail (a load counts from one),
// RS_FAULT_ALLOC=load_scratch the scratch of a load on the device.
struct DevReq {
    void **p;
    size_t bytes;
};
// Buffers are laid out at multiples of 256 bytes.
static size_t slab_part(const DevReq &r) { return (std::max<size_t>(r.bytes, 16) + 255) / 256 * 256; }
template <size_t N>
static size_t group_bytes(const std::array<DevReq, N> &reqs) {
    size_t total = 0;
    for (const DevReq &r : reqs) total += slab_part(r);
    return total;
}
// Buffers that live and die together share one device allocation (its base in
// *slab, if wanted): a graph's sixty buffers cost 75 us each to free and 20 us
// to allocate one by one.  On an error no pointer is changed.
static hipError_t dev_alloc_group(rs_graph *g, const DevReq *reqs, size_t n, void **slab = nullptr) {
    const char *f = std::getenv("RS_FAULT_ALLOC");
    size_t total = 0;
    for (size_t i = 0; i < n; ++i) {
        total += slab_part(reqs[i]);
        if (f && std::atoll(f) == ++g->n_requests) return hipErrorOutOfMemory;
    }
    char *base = nullptr;
    const hipError_t e = hipMalloc((void **)&base, total);
    if (e != hipSuccess) return e;
    try {
        g->allocations.push_back({base, total});
    } catch (...) {
        (void)hipFree(base);
        return hipErrorOutOfMemory;
    }
    g->dev_bytes += (int64_t)total;
    if (slab) *slab = base;
    for (size_t i = 0; i < n; ++i) {
        *reqs[i].p = base;
        base += slab_part(reqs[i]);
    }
    return e;
}
static hipError_t dev_alloc(rs_graph *g, void **p, size_t bytes) {
    const DevReq r = {p, bytes};
    return dev_alloc_group(g, &r, 1);
}

// Free one buffer of the graph (the stream must be idle).
static void dev_free(rs_graph *g, void **p) {
    if (!*p) return;
    for (size_t i = 0; i < g->allocations.size(); ++i)
        if (g->allocations[i].first == *p) {
            g->dev_bytes -= (int64_t)g->allocations[i].second;
            g->allocations.erase(g->allocations.begin() + (long)i);
            break;
        }
    (void)hipFree(*p);
    *p = nullptr;
}

static void release(rs_graph *g) {
    if (!g) return;
    if (g->stream) (void)hipStreamSynchronize(g->stream);
    for (auto &a : g->allocations) (void)hipFree(a.first);
    g->allocations.clear();
    if (g->hpin_own) (void)hipHostFree(g->hpin);
    if (g->pin) (void)hipHostFree(g->pin);
    g->hpin_own = false;
    g->pin = nullptr;
    g->hpin = nullptr;
    g->hpin_cap = 0;
    if (g->bpin) (void)hipHostFree(g->bpin);
    g->bpin = nullptr;
    if (g->read_host) (void)hipHostFree(g->read_host);
    g->read_host = nullptr;
    g->read_cap = 0;
    if (g->rem_buf) (void)hipFree(g->rem_buf);
    if (g->rem_host) (void)hipHostFree(g->rem_host);
    if (g->rem_ev) (void)hipEventDestroy(g->rem_ev);
    g->rem_ev = nullptr;
    if (g->reach_host) (void)hipHostFree(g->reach_host);
    g->reach_host = g->reach_cnt = nullptr;
    g->reach_comp = nullptr;
    g->reach_bits = nullptr;
    g->rem_buf = g->rem_host = nullptr;
    g->rem_cnt_host = nullptr;
    g->rem_cap = g->rem_host_cap = 0;
    for (hipEvent_t e : g->timing.pool) (void)hipEventDestroy(e);
    for (auto &pe : g->timing.pending) {
        (void)hipEventDestroy(pe.second.first);
        (void)hipEventDestroy(pe.second.second);
    }
    g->timing.pool.clear();
    g->timing.pending.clear();
    if (g->own_stream && g->stream) (void)hipStreamDestroy(g->stream);
    g->stream = nullptr;
}

// ------------------------------------------------------------ timing
static hipEvent_t take_event(rs_graph *g) {
    hipEvent_t e = nullptr;
    if (!g->timing.pool.empty()) {
        e = g->timing.pool.back();
        g->timing.pool.pop_back();
    } else if (hipEventCreate(&e) != hipSuccess) {
        e = nullptr;
    }
    return e;
}

void timing_begin(rs_graph *g, int kid, hipEvent_t *ev) {
    (void)kid;
    *ev = nullptr;
    if (!g->timing.on) return;
    *ev = take_event(g);
    if (*ev) (void)hipEventRecord(*ev, g->stream);
}

void timing_end(rs_graph *g, int kid, hipEvent_t ev) {
    if (!g->timing.on || !ev) return;
    hipEvent_t e2 = take_event(g);
    if (!e2) {
        g->timing.pool.push_back(ev);
        return;
    }
    (void)hipEventRecord(e2, g->stream);
    g->timing.pending.push_back({kid, {ev, e2}});
}

// ------------------------------------------------------------ validation
template <class OffIn>
static rs_status validate_graph(int64_t n, int64_t nnz, const OffIn *off, const int32_t *col, const int32_t *lab) {
    if ((int64_t)off[0] != 0) return fail(RS_ERR_GRAPH, "row_offsets[0] != 0");
    for (int64_t u = 0; u < n; ++u)
        if ((int64_t)off[u + 1] < (int64_t)off[u])
            return fail(RS_ERR_GRAPH, "row_offsets decrease at vertex " + std::to_string(u));
    if ((int64_t)off[n] != nnz) return fail(RS_ERR_GRAPH, "row_offsets[n] != nnz");
    for (int64_t u = 0; u < n; ++u)
        if (lab[u] < 0) return fail(RS_ERR_GRAPH, "negative label at vertex " + std::to_string(u));
    for (int64_t i = 0; i < nnz; ++i)
        if (col[i] < 0 || col[i] >= n) return fail(RS_ERR_RANGE, "neighbour id out of range at entry " + std::to_string(i));
    std::atomic<int> bad{0};
    std::atomic<int64_t> bad_at{-1};
    parallel_for(n, 4096, [&](int64_t lo, int64_t hi) {
        for (int64_t u = lo; u < hi && !bad.load(std::memory_order_relaxed); ++u) {
            const int64_t b = (int64_t)off[u], e = (int64_t)off[u + 1];
            for (int64_t i = b; i < e; ++i) {
                const int32_t v = col[i];
                int why = 0;
                if (v < 0 || v >= n)
                    why = 3;
                else if (v == u)
                    why = 1;
                else if (i > b && col[i - 1] >= v)
                    why = 2;
                else {
                    const int32_t *rb = col + (int64_t)off[v], *re = col + (int64_t)off[v + 1];
                    const int32_t *it = std::lower_bound(rb, re, (int32_t)u);
                    if (it == re || *it != (int32_t)u) why = 4;
                }
                if (why) {
                    int expected = 0;
                    if (bad.compare_exchange_strong(expected, why)) bad_at.store(u);
                    return;
                }
            }
        }
    });
    switch (bad.load()) {
        case 0: return RS_OK;
        case 1: return fail(RS_ERR_GRAPH, "self-loop at vertex " + std::to_string(bad_at.load()));
        case 2: return fail(RS_ERR_GRAPH, "row not strictly ascending (unsorted or duplicate) at vertex " +
                                              std::to_string(bad_at.load()));
        case 3: return fail(RS_ERR_RANGE, "neighbour id out of range in row " + std::to_string(bad_at.load()));
        default: return fail(RS_ERR_GRAPH, "asymmetric adjacency at vertex " + std::to_string(bad_at.load()));
    }
}

// ------------------------------------------------------------ load
// The static schedule of a graph under one Tiling: row tiles and hub rows,
// score tiles, score hubs and their chunks, and the blocks of each vertex.
struct HostTiles {
    std::vector<int2> rtv, stiles, schunk;
    std::vector<RowTile> rtiles;
    std::vector<int32_t> vrowb, vscore;  // the row block and score unit of each vertex
    std::vector<int32_t> rhubs, shubs, sfirst;
    std::vector<int32_t> gblk_off, gblk;  // batches: the row blocks of each graph
    int n_chunks_lds = 0;
    int n_hubs_lds = 0;  // score hubs whose foreign list fits in LDS (listed first)
};

struct HostGraph : HostTiles {
    std::vector<int64_t> off;   // internal offsets
    std::vector<int32_t> col;   // internal rows
    std::vector<int32_t> lab;   // internal community per internal vertex
    std::vector<int32_t> new2old, old2new, comm2orig;
    std::vector<int64_t> oo;
    std::vector<int32_t> goff, fcol, outl, cstart;
};

// Greedy cut of the vertex sequence into tiles of consecutive vertices: a
// tile closes when the next vertex would push its weight past wcap or its
// vertex count past vcap, and at every vertex listed in cuts (ascending).  A
// vertex heavier than wcap is a hub.
static void cut_tiles(int64_t n, const std::vector<int64_t> &weight, int64_t wcap, int64_t vcap,
                      std::vector<int2> &tiles, std::vector<int32_t> &hubs,
                      const std::vector<int64_t> &cuts = std::vector<int64_t>()) {
    int64_t lo = 0, w = 0;
    size_t ci = 0;
    for (int64_t v = 0; v < n; ++v) {
        if (ci < cuts.size() && cuts[ci] <= v) {
            while (ci < cuts.size() && cuts[ci] <= v) ++ci;
            if (v > lo) tiles.push_back(make_int2((int)lo, (int)v));
            lo = v;
            w = 0;
        }
        const int64_t x = weight[v];
        if (x > wcap) {
            if (v > lo) tiles.push_back(make_int2((int)lo, (int)v));
            hubs.push_back((int32_t)v);
            lo = v + 1;
            w = 0;
            continue;
        }
        if (w + x > wcap || v - lo == vcap) {
            tiles.push_back(make_int2((int)lo, (int)v));
            lo = v;
            w = 0;
        }
        w += x;
    }
    if (n > lo) tiles.push_back(make_int2((int)lo, (int)n));
}

// Cut the static schedule for the tiling T from the internal row offsets,
// each vertex's row capacity and load-time foreign degree (vstart: a batch's
// graph starts; tiles never span two graphs).
static void cut_all(int64_t n, const std::vector<int64_t> &off, const std::vector<int64_t> &cap,
                    const std::vector<int64_t> &fgn, const std::vector<int64_t> &vstart, const Tiling &T,
                    HostTiles &H) {
    H = HostTiles();
    cut_tiles(n, cap, T.row_entries, T.row_vertices, H.rtv, H.rhubs, vstart);
    H.rtiles.resize(H.rtv.size());
    for (size_t t = 0; t < H.rtv.size(); ++t) {
        RowTile &rt = H.rtiles[t];
        rt.v0 = H.rtv[t].x;
        rt.v1 = H.rtv[t].y;
        rt.e0 = off[rt.v0];
        rt.te = (int)(off[rt.v1] - off[rt.v0]);
        rt.pad = 0;
    }
    cut_tiles(n, fgn, T.score_pairs, T.score_vertices, H.stiles, H.shubs);
    // a score hub's pairs are processed kScoreTileP at a time, one chunk per workgroup
    // hubs whose foreign list fits in LDS are listed (and chunked) first
    std::stable_partition(H.shubs.begin(), H.shubs.end(), [&](int32_t v) { return fgn[v] <= T.hub_list; });
    H.sfirst.assign(1, 0);
    H.n_chunks_lds = 0;
    H.n_hubs_lds = 0;
    for (size_t h = 0; h < H.shubs.size(); ++h) {
        if (fgn[H.shubs[h]] <= T.hub_list) H.n_hubs_lds = (int)h + 1;
        const int64_t nch = (fgn[H.shubs[h]] + kScoreTileP - 1) / kScoreTileP;
        for (int64_t c = 0; c < nch; ++c) H.schunk.push_back(make_int2((int)h, (int)c));
        H.sfirst.push_back((int32_t)H.schunk.size());
        if (fgn[H.shubs[h]] <= T.hub_list) H.n_chunks_lds = (int)H.schunk.size();
    }
    // the block of the full launch that handles each vertex: hubs take
    // the first blocks, tile t of XCD x = t / per runs at block
    // hubs + 8 (t % per) + ((x - hubs) mod 8) (the inverse of the
    // kernels' block-to-tile map)
    auto tile_block = [](int64_t t, int64_t n_tiles, int64_t hubs) {
        const int64_t per = (n_tiles + 7) / 8, x = t / per, q = t % per;
        return (int32_t)(hubs + 8 * q + (((x - hubs) % 8 + 8) % 8));
    };
    H.vrowb.assign(n, 0);
    for (size_t h = 0; h < H.rhubs.size(); ++h) H.vrowb[H.rhubs[h]] = (int32_t)h;
    for (size_t t = 0; t < H.rtv.size(); ++t)
        for (int v = H.rtv[t].x; v < H.rtv[t].y; ++v)
            H.vrowb[v] = tile_block((int64_t)t, (int64_t)H.rtv.size(), (int64_t)H.rhubs.size());
    H.vscore.assign(n, 0);
    for (size_t h = 0; h < H.shubs.size(); ++h) H.vscore[H.shubs[h]] = -1 - (int32_t)h;
    for (size_t t = 0; t < H.stiles.size(); ++t)
        for (int v = H.stiles[t].x; v < H.stiles[t].y; ++v)
            H.vscore[v] = tile_block((int64_t)t, (int64_t)H.stiles.size(), (int64_t)H.n_chunks_lds);
    if (!vstart.empty()) {
        // each row block lies in one graph (tiles are cut at the graph
        // starts): list the blocks of every graph, for its w_max
        const int64_t G = (int64_t)vstart.size() - 1;
        auto graph_of = [&](int64_t v) {
            return (int64_t)(std::upper_bound(vstart.begin(), vstart.end(), v) - vstart.begin()) - 1;
        };
        std::vector<std::pair<int32_t, int32_t>> bg;  // (graph, block)
        for (size_t h = 0; h < H.rhubs.size(); ++h) bg.emplace_back((int32_t)graph_of(H.rhubs[h]), (int32_t)h);
        for (size_t t = 0; t < H.rtv.size(); ++t)
            bg.emplace_back((int32_t)graph_of(H.rtv[t].x),
                            tile_block((int64_t)t, (int64_t)H.rtv.size(), (int64_t)H.rhubs.size()));
        std::sort(bg.begin(), bg.end());
        H.gblk_off.assign(G + 1, 0);
        H.gblk.resize(bg.size());
        for (size_t i = 0; i < bg.size(); ++i) {
            ++H.gblk_off[bg[i].first + 1];
            H.gblk[i] = bg[i].second;
        }
        for (int64_t gi = 0; gi < G; ++gi) H.gblk_off[gi + 1] += H.gblk_off[gi];
    }
}

// vstart: for a batch, the first vertex of each graph and n (a graph's
// vertices keep one contiguous id range through the renumbering, since its
// labels are ranked above those of the graphs before it); empty otherwise.
template <class OffIn>
static rs_status build_internal(int64_t n, int64_t nnz, const OffIn *off, const int32_t *col, const int32_t *lab,
                                const std::vector<int64_t> &vstart, HostGraph &H) {
    try {
        // communities: ascending caller label -> internal id 0..k-1
        H.comm2orig.assign(lab, lab + n);
        std::sort(H.comm2orig.begin(), H.comm2orig.end());
        H.comm2orig.erase(std::unique(H.comm2orig.begin(), H.comm2orig.end()), H.comm2orig.end());
        const int64_t k = (int64_t)H.comm2orig.size();
        std::vector<int32_t> cid(n);
        parallel_for(n, 1 << 16, [&](int64_t lo, int64_t hi) {
            for (int64_t v = lo; v < hi; ++v)
                cid[v] = (int32_t)(std::lower_bound(H.comm2orig.begin(), H.comm2orig.end(), lab[v]) -
                                   H.comm2orig.begin());
        });
        // vertices: counting sort by community, stable in caller id
        std::vector<int64_t> start(k + 1, 0);
        for (int64_t v = 0; v < n; ++v) ++start[cid[v] + 1];
        for (int64_t c = 0; c < k; ++c) start[c + 1] += start[c];
        H.new2old.resize(n);
        H.old2new.resize(n);
        H.lab.resize(n);
        {
            std::vector<int64_t> fill(start.begin(), start.end() - 1);
            for (int64_t v = 0; v < n; ++v) {
                const int64_t nv = fill[cid[v]]++;
                H.new2old[nv] = (int32_t)v;
                H.old2new[v] = (int32_t)nv;
                H.lab[nv] = cid[v];
            }
        }
        // rows in internal ids, sorted
        H.off.assign(n + 1, 0);
        for (int64_t nv = 0; nv < n; ++nv) {
            const int64_t v = H.new2old[nv];
            H.off[nv + 1] = H.off[nv] + ((int64_t)off[v + 1] - (int64_t)off[v]);
        }
        H.col.resize(nnz);
        parallel_for(n, 1024, [&](int64_t lo, int64_t hi) {
            for (int64_t nv = lo; nv < hi; ++nv) {
                const int64_t v = H.new2old[nv];
                const int64_t b = (int64_t)off[v], e = (int64_t)off[v + 1];
                int32_t *dst = H.col.data() + H.off[nv];
                for (int64_t i = b; i < e; ++i) dst[i - b] = H.old2new[col[i]];
                std::sort(dst, dst + (e - b));
            }
        });
        // tiles: row tiles bound the row capacity, score tiles the foreign
        // entries (own-community neighbours form the id range of the community)
        std::vector<int64_t> cap(n), fgn(n);
        parallel_for(n, 4096, [&](int64_t lo, int64_t hi) {
            for (int64_t nv = lo; nv < hi; ++nv) {
                const int32_t *b = H.col.data() + H.off[nv], *e = H.col.data() + H.off[nv + 1];
                const int32_t c = H.lab[nv];
                const int64_t own = std::lower_bound(b, e, (int32_t)start[c + 1]) - std::lower_bound(b, e, (int32_t)start[c]);
                cap[nv] = e - b;
                fgn[nv] = (e - b) - own;
            }
        });
        // out-lists: foreign neighbours of higher rank (foreign degree, id)
        H.oo.assign(n + 1, 0);
        auto higher = [&](int64_t x, int32_t y) { return fgn[y] > fgn[x] || (fgn[y] == fgn[x] && y > x); };
        auto foreign = [&](int64_t x, int32_t y) { return H.lab[y] != H.lab[x]; };
        parallel_for(n, 4096, [&](int64_t lo, int64_t hi) {
            for (int64_t x = lo; x < hi; ++x) {
                int64_t c = 0;
                for (int64_t j = H.off[x]; j < H.off[x + 1]; ++j) {
                    const int32_t y = H.col[j];
                    if (foreign(x, y) && higher(x, y)) ++c;
                }
                H.oo[x + 1] = c;
            }
        });
        for (int64_t x = 0; x < n; ++x) H.oo[x + 1] += H.oo[x];
        H.outl.resize(H.oo[n]);
        parallel_for(n, 4096, [&](int64_t lo, int64_t hi) {
            for (int64_t x = lo; x < hi; ++x) {
                int64_t o = H.oo[x];
                for (int64_t j = H.off[x]; j < H.off[x + 1]; ++j) {
                    const int32_t y = H.col[j];
                    if (foreign(x, y) && higher(x, y)) H.outl[o++] = y;
                }
            }
        });
        // link slots: u's foreign entries in row order (the links themselves
        // are built on the device)
        if (H.oo[n] > (int64_t)INT32_MAX) return fail(RS_ERR_RANGE, "out-lists exceed 32-bit offsets");
        if (H.oo[n] >= (int64_t)1 << 30)
            return fail(RS_ERR_RANGE, "more than 2^30 edges between communities (slots are 32-bit)");
        H.goff.assign(n + 1, 0);
        for (int64_t x = 0; x < n; ++x) H.goff[x + 1] = H.goff[x] + (int32_t)fgn[x];
        H.fcol.resize(H.goff[n]);
        parallel_for(n, 4096, [&](int64_t lo, int64_t hi) {
            for (int64_t x = lo; x < hi; ++x) {
                int32_t o = H.goff[x];
                for (int64_t j = H.off[x]; j < H.off[x + 1]; ++j)
                    if (foreign(x, H.col[j])) H.fcol[o++] = H.col[j];
            }
        });
        H.cstart.resize(k + 1);
        for (int64_t c = 0; c <= k; ++c) H.cstart[c] = (int32_t)start[c];
        cut_all(n, H.off, cap, fgn, vstart, Tiling(), H);
    } catch (const std::bad_alloc &) {
        return fail(RS_ERR_NOMEM, "host allocation failed while renumbering the graph");
    }
    return RS_OK;
}

static int rows_grid(const HostTiles &H) { return tile_grid((int)H.rhubs.size(), (int)H.rtiles.size()); }
static int score_grid(const HostTiles &H) { return tile_grid((int)H.schunk.size(), (int)H.stiles.size()); }

// The schedule's device arrays.
static auto tile_reqs(DeviceGraph &D, int64_t n_out, const HostTiles &H) {
    const size_t N = (size_t)std::max<int64_t>(D.n, 1);
    const size_t nch = std::max<size_t>(H.schunk.size(), 1);
    const size_t nrt = std::max<size_t>(H.rtiles.size(), 1), nrh = std::max<size_t>(H.rhubs.size(), 1);
    const size_t nst = std::max<size_t>(H.stiles.size(), 1), nsh = std::max<size_t>(H.shubs.size(), 1);
    const size_t gr = (size_t)std::max(rows_grid(H), 1), gs = (size_t)std::max(score_grid(H), 1);
    return std::array{
        DevReq{(void **)&D.rtiles, sizeof(RowTile) * nrt},
        DevReq{(void **)&D.rhubs, 4 * nrh},
        DevReq{(void **)&D.stiles, sizeof(int2) * nst},
        DevReq{(void **)&D.shubs, 4 * nsh},
        DevReq{(void **)&D.shub_first, 4 * (nsh + 1)},
        DevReq{(void **)&D.shub_chunk, sizeof(int2) * nch},
        DevReq{(void **)&D.hub_part, sizeof(HubPart) * nch},
        DevReq{(void **)&D.rflag, gr},
        DevReq{(void **)&D.cflag, nch},
        DevReq{(void **)&D.hflag, nsh},
        DevReq{(void **)&D.rlist, 4 * gr},
        DevReq{(void **)&D.slist, 4 * gs},
        DevReq{(void **)&D.hlist, 4 * nch},
        DevReq{(void **)&D.part_rows, sizeof(RowPart) * gr},
        DevReq{(void **)&D.wmax_part, 8 * gr},
        DevReq{(void **)&D.vrowb, 4 * N},
        DevReq{(void **)&D.vscore, 4 * N},
        DevReq{(void **)&D.sown, (size_t)std::max<int64_t>(2 * n_out, 1)},
        DevReq{(void **)&D.hfilter, 4 * (size_t)kFilterWords * std::max<size_t>(H.shubs.size() - H.n_hubs_lds, 1)}
    };
}

// Allocate and fill the schedule's device arrays: tiles and hubs, the
// per-block partials, the incremental re-score's unit flags and lists, and each
// vertex's row block and score unit.  Leaves the copies queued on the graph's
// stream, and any earlier schedule's arrays to the caller.
static rs_status upload_tiles(rs_graph *g, const HostTiles &H) {
    DeviceGraph &D = g->d;
    const auto reqs = tile_reqs(D, g->n_out, H);
    hipError_t e = dev_alloc_group(g, reqs.data(), reqs.size(), &g->tile_slab);
    if (e != hipSuccess) return hip_fail(e, "device allocation");
    g->n_rtiles = (int)H.rtiles.size();
    g->n_rhubs = (int)H.rhubs.size();
    g->n_stiles = (int)H.stiles.size();
    g->n_shubs = (int)H.shubs.size();
    g->n_schunks = (int)H.schunk.size();
    g->n_schunks_lds = H.n_chunks_lds;
    g->n_shubs_lds = H.n_hubs_lds;
    g->grid_rows = rows_grid(H);
    g->grid_score = score_grid(H);
    hipStream_t s = g->stream;
    auto put = [&](void *dst, const void *src, size_t bytes) {
        if (e == hipSuccess && bytes) e = hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s);
    };
    put(D.rtiles, H.rtiles.data(), sizeof(RowTile) * H.rtiles.size());
    put(D.rhubs, H.rhubs.data(), 4 * H.rhubs.size());
    put(D.stiles, H.stiles.data(), sizeof(int2) * H.stiles.size());
    put(D.shubs, H.shubs.data(), 4 * H.shubs.size());
    put(D.shub_first, H.sfirst.data(), 4 * H.sfirst.size());
    put(D.shub_chunk, H.schunk.data(), sizeof(int2) * H.schunk.size());
    put(D.vrowb, H.vrowb.data(), 4 * H.vrowb.size());
    put(D.vscore, H.vscore.data(), 4 * H.vscore.size());
    if (e == hipSuccess) e = hipMemsetAsync(D.rflag, 0, (size_t)std::max(g->grid_rows, 1), s);
    if (e == hipSuccess) e = hipMemsetAsync(D.cflag, 0, std::max<size_t>(H.schunk.size(), 1), s);
    if (e == hipSuccess) e = hipMemsetAsync(D.hflag, 0, std::max<size_t>(H.shubs.size(), 1), s);
    return e == hipSuccess ? launch_slot_owners(g) : hip_fail(e, "schedule upload");
}

// The graph's device arrays: those sized by its vertices and entries, cleared
// where a pass expects it, and those sized by its slots (2 n_out).
static void set_sizes(DeviceGraph &D, int64_t n, int64_t nnz, int64_t k, bool wide) {
    D.n = n;
    D.nnz = nnz;
    D.k = (int32_t)k;
    D.off64 = nnz > (int64_t)INT32_MAX || wide;
}
static auto vertex_reqs(DeviceGraph &D) {
    const size_t N = (size_t)std::max<int64_t>(D.n, 1), Z = (size_t)std::max<int64_t>(D.nnz, 1);
    const size_t offb = D.off64 ? 8 : 4;
    return std::array{
        DevReq{&D.off, offb * (N + 1)},
        DevReq{(void **)&D.deg, 4 * N},
        DevReq{(void **)&D.col, 4 * Z},
        DevReq{(void **)&D.clab, 4 * Z},
        DevReq{(void **)&D.lab, 4 * N},
        DevReq{(void **)&D.new2old, 4 * N},
        DevReq{(void **)&D.alive, N},
        DevReq{(void **)&D.oo, 8 * (N + 1)},
        DevReq{(void **)&D.goff, 4 * (N + 1)},
        DevReq{(void **)&D.cstart, 4 * ((size_t)D.k + 1)},
        DevReq{(void **)&D.wpart, 8 * (size_t)kWorkBlocks},
        DevReq{(void **)&D.tables, table_bytes()},
        DevReq{(void **)&D.raw, 8 * N},
        DevReq{(void **)&D.vmark, 4 * N},
        DevReq{(void **)&D.elist, 4 * N},
        DevReq{(void **)&D.ucnt, 4 * (size_t)kUnitRows * kUnitGroups},
        DevReq{(void **)&D.abin, 4 * N},
        DevReq{(void **)&D.echunk, sizeof(int2) * (N + Z / 64 + 1)},
        DevReq{(void **)&D.ictr, 8 * (size_t)kIcCount},
        DevReq{(void **)&D.ictr_next, 8 * (size_t)kIcCount},
        DevReq{(void **)&D.wblk, 8 * 64},
        DevReq{(void **)&D.wticket, 8},
        DevReq{(void **)&D.meta, sizeof(VMeta) * N},
        DevReq{(void **)&D.wown, 8 * N},
        DevReq{(void **)&D.av, 8 * N},
        DevReq{(void **)&D.R, 8 * N},
        DevReq{(void **)&D.tI, 8 * N},
        DevReq{(void **)&D.tII, 8 * N},
        DevReq{(void **)&D.ctr, sizeof(DevCounters)},
        DevReq{(void **)&D.thist, 4 * (size_t)kTopkBins},
        DevReq{(void **)&D.thist_c, 4 * 256},
        DevReq{(void **)&D.tstate, sizeof(TopkState)},
        DevReq{(void **)&D.tfinal, sizeof(TopkKey) * N},
        DevReq{(void **)&D.ttie, sizeof(TopkKey) * N},
        DevReq{(void **)&D.ttie2, sizeof(TopkKey) * N},
        DevReq{(void **)&D.tout_ids, 4 * N},
        DevReq{(void **)&D.tout_sc, 8 * N},
        DevReq{(void **)&D.scratch_d, 8 * N},
        DevReq{(void **)&D.tblk, 16 + 16 * N},
        DevReq{(void **)&D.scratch_u, 8 * 8}
    };
}
static auto slot_reqs(DeviceGraph &D, int64_t n_out) {
    const size_t NX = std::max<size_t>(2 * (size_t)n_out, 1), NO = std::max<size_t>((size_t)n_out, 1);
    return std::array{
        DevReq{(void **)&D.fcol, 4 * NX},
        DevReq{(void **)&D.prec, sizeof(PairRec) * NX},
        DevReq{(void **)&D.val2, 8 * NX},
        DevReq{(void **)&D.plink, sizeof(PairLink) * NX},
        DevReq{(void **)&D.outl, 4 * NO},
        DevReq{(void **)&D.oe, sizeof(OutEnt) * NO}
    };
}

static rs_status alloc_vertices(rs_graph *g, int64_t n, int64_t nnz, int64_t k) {
    DeviceGraph &D = g->d;
    set_sizes(D, n, nnz, k, g->wide_offsets);
    const size_t N = (size_t)std::max<int64_t>(n, 1);
    const auto reqs = vertex_reqs(D);
    hipError_t e = dev_alloc_group(g, reqs.data(), reqs.size());
    if (e != hipSuccess) return hip_fail(e, "device allocation");
    hipStream_t s = g->stream;
    e = hipMemsetAsync(D.alive, 1, N, s);
    if (e == hipSuccess) e = hipMemsetAsync(D.vmark, 0, 4 * N, s);
    if (e == hipSuccess) e = hipMemsetAsync(D.thist, 0, 4 * (size_t)kTopkBins, s);
    if (e == hipSuccess) e = hipMemsetAsync(D.thist_c, 0, 4 * 256, s);
    if (e == hipSuccess) e = hipMemsetAsync(D.ctr, 0, sizeof(DevCounters), s);
    if (e == hipSuccess) e = hipMemsetAsync(D.wticket, 0, 8, s);
    if (e == hipSuccess) e = hipMemsetAsync(D.tstate, 0, sizeof(TopkState), s);
    if (e == hipSuccess) e = hipMemsetAsync(D.ictr, 0, 8 * (size_t)kIcCount, s);
    if (e == hipSuccess) e = hipMemsetAsync(D.ictr_next, 0, 8 * (size_t)kIcCount, s);
    return e == hipSuccess ? RS_OK : hip_fail(e, "graph upload");
}

static rs_status alloc_slots(rs_graph *g, int64_t n_out) {
    g->n_out = n_out;
    const auto reqs = slot_reqs(g->d, n_out);
    const hipError_t e = dev_alloc_group(g, reqs.data(), reqs.size());
    return e == hipSuccess ? RS_OK : hip_fail(e, "device allocation");
}

// The row offsets in the device's width.
static hipError_t put_offsets(rs_graph *g, const std::vector<int64_t> &off, std::vector<int32_t> &off32) {
    const size_t n1 = off.size();
    if (g->d.off64) return hipMemcpyAsync(g->d.off, off.data(), 8 * n1, hipMemcpyHostToDevice, g->stream);
    off32.resize(n1);
    parallel_for((int64_t)n1, 1 << 18, [&](int64_t lo, int64_t hi) {
        for (int64_t v = lo; v < hi; ++v) off32[v] = (int32_t)off[v];
    });
    return hipMemcpyAsync(g->d.off, off32.data(), 4 * n1, hipMemcpyHostToDevice, g->stream);
}

// The handle's pinned memory, in one allocation (64 bytes or 16 KB: 12 us to make
// and 12 to free), and its event.  A batch takes no removals and has its own
// top-k.
static rs_status alloc_pinned(rs_graph *g) {
    constexpr size_t kCounts = 64;
    static_assert(sizeof(RemovalCounts) <= kCounts, "the counts' place");
    hipError_t e = hipSuccess;
    if (!g->pin && g->n_graphs == 0) {
        e = hipHostMalloc((void **)&g->pin, kCounts + 16 + 16 * (size_t)kPinK, hipHostMallocDefault);
        if (e != hipSuccess) {
            g->pin = nullptr;
            return hip_fail(e, "pinned counters");
        }
        g->rem_cnt_host = (RemovalCounts *)g->pin;
        g->hpin = g->pin + kCounts;
        g->hpin_cap = kPinK;
    }
    if (!g->rem_ev && g->n_graphs == 0) {
        e = hipEventCreateWithFlags(&g->rem_ev, hipEventDisableTiming);
        if (e != hipSuccess) {
            g->rem_ev = nullptr;
            return hip_fail(e, "removal event");
        }
    }
    return RS_OK;
}

// What follows once the rows, slots and out-lists are in place: the schedule
// (cut in H), the links and the out-list entries' leaders.
static rs_status finish_load(rs_graph *g, const HostGraph &H) {
    DeviceGraph &D = g->d;
    rs_status st = upload_tiles(g, H);
    if (st == RS_OK) st = launch_tables(g);
    if (st == RS_OK) st = launch_zero_u64(g, D.scratch_u, 1);
    if (st == RS_OK) st = launch_links(g, D.scratch_u);
    if (st != RS_OK) return st;
    unsigned long long walk = 0;
    hipError_t e = hipMemcpyAsync(&walk, D.scratch_u, 8, hipMemcpyDeviceToHost, g->stream);
    if (e == hipSuccess) st = launch_out_entries(g);
    if (st == RS_OK) st = alloc_pinned(g);                  // (while the device works)
    const hipError_t es = hipStreamSynchronize(g->stream);  // (on an error too: walk is this frame's)
    if (st != RS_OK) return st;
    if (e == hipSuccess) e = es;
    if (e != hipSuccess) return hip_fail(e, "pair-slot map");
    // The type-II values by slot cost each slot its record and neighbour once
    // more; the pairs walking the runs themselves cost a gather a step, by one
    // lane.  Passes by slot against walks, with half the steps (walk) as a share
    // of the slots: 0.07 164 against 156 us (n = 1 million, mean degree 20), 0.17
    // 126 against 118 (n = 300,000), 0.22 387 against 372, 0.27 594 against 568
    // (n = 1 million, mean degree 30, mixing 0.3), 0.39 99 against 95 (n =
    // 100,000, mean degree 40), 0.43 340 against 383 (n = 1 million, hubs of
    // 30,000), 0.48 246 against 256 (n = 300,000), and, with earlier kernels,
    // 1.06 1,818 against 2,675 (n = 3 million, mean degree 30) and 1.21 686
    // against 776 (n = 150,000, mean degree 71).  Below the line of a quarter
    // the walks are faster; up to 0.4 the values by slot lose 4 to 6 %, but
    // hubs' long runs are never left to one lane.
    g->type2_by_slot = 4 * walk >= 2 * (unsigned long long)g->n_out;
    g->n_alive = D.n;
    return RS_OK;
}

// keep: H stays intact for later uploads (its host maps are copied, not moved)
static rs_status upload(rs_graph *g, HostGraph &H, int64_t n, int64_t nnz, bool keep = false) {
    DeviceGraph &D = g->d;
    rs_status st = alloc_vertices(g, n, nnz, (int64_t)H.comm2orig.size());
    if (st == RS_OK) st = alloc_slots(g, (int64_t)H.outl.size());
    if (st != RS_OK) return st;
    std::vector<int32_t> off32, deg;
    hipError_t e;
    try {
        deg.resize(n);
        for (int64_t v = 0; v < n; ++v) deg[v] = (int32_t)(H.off[v + 1] - H.off[v]);
        e = put_offsets(g, H.off, off32);
    } catch (const std::bad_alloc &) {
        return fail(RS_ERR_NOMEM, "host staging of the upload");
    }
    auto put = [&](void *dst, const void *src, size_t bytes) {
        if (e == hipSuccess && bytes) e = hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, g->stream);
    };
    put(D.deg, deg.data(), 4 * (size_t)n);
    put(D.col, H.col.data(), 4 * (size_t)nnz);
    put(D.lab, H.lab.data(), 4 * (size_t)n);
    put(D.new2old, H.new2old.data(), 4 * (size_t)n);
    put(D.oo, H.oo.data(), 8 * H.oo.size());
    put(D.goff, H.goff.data(), 4 * H.goff.size());
    put(D.fcol, H.fcol.data(), 4 * H.fcol.size());
    put(D.cstart, H.cstart.data(), 4 * H.cstart.size());
    put(D.outl, H.outl.data(), 4 * H.outl.size());
    const hipError_t es = hipStreamSynchronize(g->stream);  // (on an error too: the staging is this frame's)
    if (e == hipSuccess) e = es;
    if (e != hipSuccess) return hip_fail(e, "graph upload");
    st = launch_col_labels(g);  // each entry's neighbour community
    if (st == RS_OK) st = finish_load(g, H);
    if (st != RS_OK) return st;
    if (keep) {
        try {
            g->h_new2old = H.new2old;
            g->h_old2new = H.old2new;
            g->h_comm2orig = H.comm2orig;
        } catch (const std::bad_alloc &) {
            return fail(RS_ERR_NOMEM, "host maps");
        }
    } else {
        g->h_new2old.swap(H.new2old);
        g->h_old2new.swap(H.old2new);
        g->h_comm2orig.swap(H.comm2orig);
    }
    return RS_OK;
}

// ------------------------------------------------------------ load on the device
// The vertices' renumbering: communities by ascending label, a stable counting
// sort of the vertices by community (in chunks, one thread each, when there are
// enough vertices for the communities), and the internal row offsets.
// False: a negative label, decreasing offsets or a row that no simple graph has
// (the host's checks say which).
template <class OffIn>
static bool renumber(int64_t n, const OffIn *off, const int32_t *lab, HostGraph &H,
                     std::vector<int64_t> &cap) {
    std::atomic<bool> ok{true};
    std::atomic<int32_t> top{0};
    parallel_for(n, 1 << 16, [&](int64_t lo, int64_t hi) {
        int32_t m = 0;
        bool good = true;
        for (int64_t v = lo; v < hi; ++v) {
            const int64_t len = (int64_t)off[v + 1] - (int64_t)off[v];
            good = good && lab[v] >= 0 && len >= 0 && len < n;
            m = std::max(m, lab[v]);
        }
        if (!good) ok.store(false);
        int32_t t = top.load();
        while (m > t && !top.compare_exchange_weak(t, m)) {
        }
    });
    if (!ok.load()) return false;
    // communities: labels up to a few times n are counted, others sorted
    const int64_t span = (int64_t)top.load() + 1;
    std::vector<int32_t> rank, cid;
    const bool dense = span <= 4 * n + 65536;
    if (dense) {
        rank.assign(span, 0);
        for (int64_t v = 0; v < n; ++v) rank[lab[v]] = 1;
        for (int64_t c = 0, r = 0; c < span; ++c) {
            if (!rank[c]) continue;
            H.comm2orig.push_back((int32_t)c);
            rank[c] = (int32_t)r++;
        }
    } else {
        H.comm2orig.assign(lab, lab + n);
        std::sort(H.comm2orig.begin(), H.comm2orig.end());
        H.comm2orig.erase(std::unique(H.comm2orig.begin(), H.comm2orig.end()), H.comm2orig.end());
    }
    const int64_t k = (int64_t)H.comm2orig.size();
    const int64_t T = n >= (1 << 17) && k <= (1 << 16) ? 8 : 1, per = (n + T - 1) / T;
    cid.resize(n);
    std::vector<int64_t> at((size_t)(T * k), 0);  // [chunk][community]: counts, then places
    parallel_for(T, 1, [&](int64_t t0, int64_t t1) {
        for (int64_t t = t0; t < t1; ++t) {
            int64_t *c = at.data() + t * k;
            for (int64_t v = t * per; v < std::min(n, (t + 1) * per); ++v) {
                cid[v] = dense ? rank[lab[v]]
                               : (int32_t)(std::lower_bound(H.comm2orig.begin(), H.comm2orig.end(), lab[v]) -
                                           H.comm2orig.begin());
                ++c[cid[v]];
            }
        }
    });
    H.cstart.resize(k + 1);
    int64_t s = 0;
    for (int64_t c = 0; c < k; ++c) {
        H.cstart[c] = (int32_t)s;
        for (int64_t t = 0; t < T; ++t) {
            const int64_t x = at[t * k + c];
            at[t * k + c] = s;
            s += x;
        }
    }
    H.cstart[k] = (int32_t)s;
    H.new2old.resize(n);
    H.old2new.resize(n);
    H.lab.resize(n);
    cap.resize(n);
    parallel_for(T, 1, [&](int64_t t0, int64_t t1) {
        for (int64_t t = t0; t < t1; ++t) {
            int64_t *c = at.data() + t * k;
            for (int64_t v = t * per; v < std::min(n, (t + 1) * per); ++v) {
                const int64_t x = c[cid[v]]++;
                H.new2old[x] = (int32_t)v;
                H.old2new[v] = (int32_t)x;
                H.lab[x] = cid[v];
                cap[x] = (int64_t)off[v + 1] - (int64_t)off[v];
            }
        }
    });
    H.off.resize(n + 1);
    H.off[0] = 0;
    for (int64_t x = 0; x < n; ++x) H.off[x + 1] = H.off[x] + cap[x];
    return true;
}

// Graphs from this many entries on are built on the device, where the host
// would sort a row at a time and look up every entry's reverse: 1.6 against
// 8.1 ms with 1.8 M entries (n = 100,000), 10 against 94 ms with 18 M, 0.40
// against 1.7 ms with 62,000.  The device's way costs 0.35 ms of launches and
// waits at the least, what the host takes for some 8,000 entries (7,700: 0.32
// ms; 15,000: 0.71 ms).
constexpr int64_t kDeviceLoadMin = 1 << 13;

// *done: the graph is loaded.  Not done with RS_OK: something is wrong with
// the graph or the device, and the host's path tells what.
template <class OffIn>
static rs_status load_on_device(const rs_csr *csr, rs_graph *g, bool *done) {
    *done = false;
    const int64_t n = csr->n, nnz = csr->nnz;
    hipStream_t s = g->stream;
    std::vector<OffIn> h_off;
    std::vector<int32_t> h_lab;
    const OffIn *off = (const OffIn *)csr->row_offsets;
    const int32_t *lab = csr->labels;
    if (csr->on_device) {
        h_off.resize(n + 1);
        h_lab.resize(n);
        hipError_t e = hipMemcpy(h_off.data(), off, sizeof(OffIn) * (n + 1), hipMemcpyDeviceToHost);
        if (e == hipSuccess) e = hipMemcpy(h_lab.data(), lab, 4 * n, hipMemcpyDeviceToHost);
        if (e != hipSuccess) return hip_fail(e, "copying the device-resident input graph");
        off = h_off.data();
        lab = h_lab.data();
    }
    // nnz is trusted (the columns' size) only when the offsets agree
    if ((int64_t)off[0] != 0 || (int64_t)off[n] != nnz) return RS_OK;
    HostGraph H;  // (these outlive the copies: the scratch's end waits for the stream)
    std::vector<int64_t> cap, fgn;
    std::vector<int32_t> off32, f32, hubs;
    // scratch of the load, one allocation
    const size_t b_off = csr->on_device ? 0 : sizeof(OffIn) * (n + 1), b_col = csr->on_device ? 0 : 4 * (size_t)nnz;
    const size_t sizes[] = {b_off, b_col, 8 * (size_t)n, 4 * (size_t)n, 8 * (size_t)prefix_blocks(n), 16,
                            4 * (size_t)(nnz / load_hub_row() + 1)};
    size_t at[8] = {0};
    for (int i = 0; i < 7; ++i) at[i + 1] = at[i] + (sizes[i] + 255) / 256 * 256;
    struct Scratch {
        char *p = nullptr;
        hipStream_t s;
        ~Scratch() {
            if (p) {
                (void)hipStreamSynchronize(s);
                (void)hipFree(p);
            }
        }
    } tmp;
    tmp.s = s;
    const char *f = std::getenv("RS_FAULT_ALLOC");
    hipError_t e = f && std::strcmp(f, "load_scratch") == 0 ? hipErrorOutOfMemory : hipMalloc((void **)&tmp.p, at[7]);
    if (e != hipSuccess) {
        tmp.p = nullptr;
        return hip_fail(e, "load scratch");
    }
    LoadArgs L;
    L.offset_bytes = (int)sizeof(OffIn);
    L.off = csr->on_device ? csr->row_offsets : tmp.p + at[0];
    L.col = csr->on_device ? csr->col : (const int32_t *)(tmp.p + at[1]);
    L.map = (int2 *)(tmp.p + at[2]);
    L.fgn = (int32_t *)(tmp.p + at[3]);
    long long *sums = (long long *)(tmp.p + at[4]);
    L.bad = (unsigned int *)(tmp.p + at[5]);
    L.hubs = (const int32_t *)(tmp.p + at[6]);
    // the columns travel while the host renumbers the vertices
    hipError_t ec = hipSuccess;
    std::thread copier;
    if (!csr->on_device) {
        const int dev = g->device;
        auto copy = [&, dev]() {
            ec = hipSetDevice(dev);
            if (ec == hipSuccess) ec = hipMemcpyAsync((void *)L.off, csr->row_offsets, b_off, hipMemcpyHostToDevice, s);
            if (ec == hipSuccess) ec = hipMemcpyAsync((void *)L.col, csr->col, b_col, hipMemcpyHostToDevice, s);
            const hipError_t es = hipStreamSynchronize(s);  // (a per-thread stream is this thread's own)
            if (ec == hipSuccess) ec = es;
        };
        try {
            copier = std::thread(copy);
        } catch (...) {
            copy();
        }
    }
    struct Join {
        std::thread &t;
        ~Join() {
            if (t.joinable()) t.join();
        }
    } join{copier};
    const bool good = renumber<OffIn>(n, off, lab, H, cap);
    for (int64_t x = 0; good && x < n; ++x)
        if (cap[x] > load_hub_row()) hubs.push_back((int32_t)x);
    if (copier.joinable()) copier.join();
    if (ec != hipSuccess) return hip_fail(ec, "graph upload");
    if (!good) return RS_OK;
    L.n_hubs = (int)hubs.size();
    rs_status st = alloc_vertices(g, n, nnz, (int64_t)H.comm2orig.size());
    if (st != RS_OK) return st;
    DeviceGraph &D = g->d;
    e = put_offsets(g, H.off, off32);
    auto put = [&](void *dst, const void *src, size_t bytes) {
        if (e == hipSuccess && bytes) e = hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s);
    };
    put(D.lab, H.lab.data(), 4 * (size_t)n);
    put(D.new2old, H.new2old.data(), 4 * (size_t)n);
    put(D.cstart, H.cstart.data(), 4 * H.cstart.size());
    put((void *)L.hubs, hubs.data(), 4 * hubs.size());
    if (e == hipSuccess) e = hipMemsetAsync(L.bad, 0, 16, s);
    if (e == hipSuccess) st = launch_load_rows(g, L);
    unsigned int bad = 0;
    f32.resize(n);
    if (e == hipSuccess && st == RS_OK) e = hipMemcpyAsync(f32.data(), L.fgn, 4 * (size_t)n, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess && st == RS_OK) e = hipMemcpyAsync(&bad, L.bad, 4, hipMemcpyDeviceToHost, s);
    const hipError_t es = hipStreamSynchronize(s);  // (on an error too: the staging is this frame's)
    if (st != RS_OK) return st;
    if (e == hipSuccess) e = es;
    if (e != hipSuccess) return hip_fail(e, "graph upload");
    if (bad) return RS_OK;
    int64_t slots = 0;
    fgn.resize(n);
    H.goff.resize(n + 1);
    for (int64_t x = 0; x < n; ++x) {
        H.goff[x] = (int32_t)slots;
        fgn[x] = f32[x];
        slots += f32[x];
        if (slots >= (int64_t)1 << 31)
            return fail(RS_ERR_RANGE, "more than 2^30 edges between communities (slots are 32-bit)");
    }
    H.goff[n] = (int32_t)slots;
    st = alloc_slots(g, slots / 2);
    if (st != RS_OK) return st;
    e = hipMemcpyAsync(D.goff, H.goff.data(), 4 * H.goff.size(), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail(e, "graph upload");
    st = launch_load_slots(g, L.fgn, sums);  // (the foreign degrees are in goff now)
    if (st != RS_OK) return st;
    cut_all(n, H.off, cap, fgn, g->h_vstart, Tiling(), H);
    g->h_gblk_off.swap(H.gblk_off);
    g->h_gblk.swap(H.gblk);
    st = finish_load(g, H);
    if (st != RS_OK) return st;
    g->h_new2old.swap(H.new2old);
    g->h_old2new.swap(H.old2new);
    g->h_comm2orig.swap(H.comm2orig);
    *done = true;
    return RS_OK;
}

// The current device, and a stream of the graph's own if the caller gave none.
static rs_status take_stream(rs_graph *g) {
    hipError_t e = hipGetDevice(&g->device);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (!g->stream) {
        e = hipStreamCreateWithFlags(&g->stream, hipStreamNonBlocking);
        if (e != hipSuccess) {
            g->stream = nullptr;
            return hip_fail(e, "hipStreamCreate");
        }
        g->own_stream = true;
    }
    return RS_OK;
}

template <class OffIn>
static rs_status load_t(const rs_csr *csr, rs_graph *g) {
    const int64_t n = csr->n, nnz = csr->nnz;
    if (nnz >= kDeviceLoadMin) {
        bool done = false;
        rs_status st = take_stream(g);
        if (st == RS_OK) {
            try {
                st = load_on_device<OffIn>(csr, g, &done);
            } catch (const std::bad_alloc &) {
                st = fail(RS_ERR_NOMEM, "host allocation failed while renumbering the graph");
            }
        }
        if (done) return RS_OK;
        // the checks below tell what is wrong with the graph or the device (or,
        // where only the load's scratch was too much, the host builds the graph)
        if (g->stream) (void)hipStreamSynchronize(g->stream);
        for (auto &a : g->allocations) (void)hipFree(a.first);
        g->allocations.clear();
        g->d = DeviceGraph();
        g->dev_bytes = 0;
        g->n_requests = 0;
        g->tile_slab = nullptr;
        (void)hipGetLastError();  // a failed allocation is not the next launch's error
        clear_error();
    }
    const OffIn *off = (const OffIn *)csr->row_offsets;
    const int32_t *col = csr->col, *lab = csr->labels;
    std::vector<OffIn> h_off;
    std::vector<int32_t> h_col, h_lab;
    if (csr->on_device) {
        try {
            h_off.resize(n + 1);
            h_col.resize(nnz);
            h_lab.resize(n);
        } catch (const std::bad_alloc &) {
            return fail(RS_ERR_NOMEM, "host staging allocation failed");
        }
        hipError_t e = hipMemcpy(h_off.data(), off, sizeof(OffIn) * (n + 1), hipMemcpyDeviceToHost);
        if (e == hipSuccess && nnz) e = hipMemcpy(h_col.data(), col, 4 * nnz, hipMemcpyDeviceToHost);
        if (e == hipSuccess && n) e = hipMemcpy(h_lab.data(), lab, 4 * n, hipMemcpyDeviceToHost);
        if (e != hipSuccess) return hip_fail(e, "copying the device-resident input graph");
        off = h_off.data();
        col = h_col.data();
        lab = h_lab.data();
    }
    rs_status st = validate_graph<OffIn>(n, nnz, off, col, lab);
    if (st != RS_OK) return st;
    HostGraph H;
    st = build_internal<OffIn>(n, nnz, off, col, lab, g->h_vstart, H);
    if (st != RS_OK) return st;
    g->h_gblk_off.swap(H.gblk_off);
    g->h_gblk.swap(H.gblk);
    st = take_stream(g);
    if (st != RS_OK) return st;
    return upload(g, H, n, nnz);
}

// A validated, renumbered and tiled host form of a graph, kept by the
// request server so that a graph evicted from device memory is reloaded by
// an upload alone.
struct Prebuilt {
    HostGraph H;
    int64_t n = 0, nnz = 0;
};

rs_status prebuild_graph(const rs_csr *csr, Prebuilt **out) {
    if (!out || !csr) return fail(RS_ERR_ARG, "csr or out is NULL");
    *out = nullptr;
    if (csr->on_device || csr->offset_bytes != 8) return fail(RS_ERR_ARG, "prebuilt graphs take host int64 offsets");
    if (csr->n < 0 || csr->nnz < 0 || csr->n > (int64_t)INT32_MAX - 1) return fail(RS_ERR_RANGE, "n or nnz out of range");
    if (!csr->row_offsets || (csr->n > 0 && !csr->labels) || (csr->nnz > 0 && !csr->col))
        return fail(RS_ERR_ARG, "null CSR array");
    const int64_t *off = (const int64_t *)csr->row_offsets;
    rs_status st = validate_graph<int64_t>(csr->n, csr->nnz, off, csr->col, csr->labels);
    if (st != RS_OK) return st;
    Prebuilt *P = new (std::nothrow) Prebuilt();
    if (!P) return fail(RS_ERR_NOMEM, "prebuilt graph");
    st = build_internal<int64_t>(csr->n, csr->nnz, off, csr->col, csr->labels, std::vector<int64_t>(), P->H);
    if (st != RS_OK) {
        delete P;
        return st;
    }
    P->n = csr->n;
    P->nnz = csr->nnz;
    *out = P;
    return RS_OK;
}

rs_status load_prebuilt(Prebuilt *P, void *hip_stream, rs_graph **out) {
    if (!P || !out) return fail(RS_ERR_ARG, "prebuilt graph or out is NULL");
    *out = nullptr;
    rs_graph *g = new (std::nothrow) rs_graph();
    if (!g) return fail(RS_ERR_NOMEM, "handle allocation failed");
    g->stream = (hipStream_t)hip_stream;
    hipError_t e = hipGetDevice(&g->device);
    rs_status st = e == hipSuccess ? RS_OK : hip_fail(e, "hipGetDevice");
    if (st == RS_OK && !g->stream) {
        e = hipStreamCreateWithFlags(&g->stream, hipStreamNonBlocking);
        if (e == hipSuccess)
            g->own_stream = true;
        else
            st = hip_fail(e, "hipStreamCreate");
    }
    if (st == RS_OK) st = upload(g, P->H, P->n, P->nnz, true);
    if (st != RS_OK) {
        std::string keep = g_err;
        release(g);
        delete g;
        g_err = keep;
        return st;
    }
    *out = g;
    return RS_OK;
}

void free_prebuilt(Prebuilt *P) { delete P; }

// (From the lists that the load itself allocates from.)
static void allocation_sizes(int64_t n, int64_t nnz, int64_t k, int64_t n_out, const HostTiles &H,
                             size_t (&bytes)[3]) {
    DeviceGraph D;
    set_sizes(D, n, nnz, k, false);
    bytes[0] = group_bytes(vertex_reqs(D));
    bytes[1] = group_bytes(slot_reqs(D, n_out));
    bytes[2] = group_bytes(tile_reqs(D, n_out, H));
}
void prebuilt_allocations(const Prebuilt *P, size_t (&bytes)[3]) {
    allocation_sizes(P->n, P->nnz, (int64_t)P->H.comm2orig.size(), (int64_t)P->H.outl.size(), P->H, bytes);
}
void least_allocations(int64_t n, int64_t nnz, size_t (&bytes)[3]) {
    allocation_sizes(n, nnz, 1, 0, HostTiles(), bytes);
}

template <class T>
static hipError_t d2h(std::vector<T> &dst, const void *src, int64_t count);

// The last pass's row facts {deg, ell, p, q} of every vertex (internal ids).
static hipError_t read_meta(rs_graph *g, std::vector<VMeta> &meta) { return d2h(meta, g->d.meta, g->d.n); }

template <class T>
static hipError_t d2h(std::vector<T> &dst, const void *src, int64_t count) {
    dst.resize(count);
    if (!count) return hipSuccess;
    return hipMemcpy(dst.data(), src, sizeof(T) * count, hipMemcpyDeviceToHost);
}

// Device results into the caller's arrays, behind what is queued on the graph's
// stream: one copy into pinned memory (at most kReadStage at a time), then the
// host threads copy on, so the caller's fresh pages are touched by all of them.
// Copies straight into pageable arrays took three times as long (n = 300,000:
// 13 MB in 4.5 ms).
struct Piece {
    void *dst;
    const void *src;
    size_t bytes;
};
constexpr size_t kReadStage = size_t(16) << 20;
static rs_status fetch_pieces(rs_graph *g, std::vector<Piece> &pieces, const char *what) {
    size_t all = 0;
    for (const Piece &p : pieces) all += (p.bytes + 63) & ~size_t(63);
    if (all == 0) return RS_OK;
    const size_t want = std::min(all, kReadStage);
    if (g->read_cap < want) {
        if (g->read_host) (void)hipHostFree(g->read_host);
        g->read_cap = 0;
        const hipError_t ea = hipHostMalloc((void **)&g->read_host, want, hipHostMallocDefault);
        if (ea != hipSuccess) {
            g->read_host = nullptr;
            return hip_fail(ea, "pinned read buffer");
        }
        g->read_cap = want;
    }
    size_t at = 0;  // the first piece not yet whole
    while (at < pieces.size()) {
        std::vector<Piece> now;  // staged this time (src: its place in the staging)
        size_t used = 0;
        hipError_t e = hipSuccess;
        for (; at < pieces.size() && used < g->read_cap && e == hipSuccess;) {
            Piece &p = pieces[at];
            const size_t b = std::min(p.bytes, g->read_cap - used);
            if (b) e = hipMemcpyAsync(g->read_host + used, p.src, b, hipMemcpyDeviceToHost, g->stream);
            now.push_back({p.dst, g->read_host + used, b});
            used = std::min(g->read_cap, used + ((b + 63) & ~size_t(63)));
            p.dst = (char *)p.dst + b;
            p.src = (const char *)p.src + b;
            p.bytes -= b;
            if (p.bytes) break;
            ++at;
        }
        const hipError_t es = hipStreamSynchronize(g->stream);
        if (e == hipSuccess) e = es;
        if (e != hipSuccess) return hip_fail(e, what);
        constexpr size_t kGrain = 256 << 10;
        std::vector<Piece> parts;
        for (const Piece &p : now)
            for (size_t o = 0; o < p.bytes; o += kGrain)
                parts.push_back({(char *)p.dst + o, (const char *)p.src + o, std::min(kGrain, p.bytes - o)});
        parallel_for((int64_t)parts.size(), 4, [&](int64_t lo, int64_t hi) {
            for (int64_t i = lo; i < hi; ++i) memcpy(parts[i].dst, parts[i].src, parts[i].bytes);
        });
    }
    return RS_OK;
}
static rs_status fetch(rs_graph *g, std::initializer_list<Piece> list, const char *what) {
    try {
        std::vector<Piece> pieces;
        for (const Piece &p : list)
            if (p.dst && p.bytes) pieces.push_back(p);
        return fetch_pieces(g, pieces, what);
    } catch (const std::bad_alloc &) {
        return fail(RS_ERR_NOMEM, what);
    }
}

static hipError_t read_offsets(rs_graph *g, std::vector<int64_t> &off) {
    const int64_t n = g->d.n;
    if (g->d.off64) return d2h(off, g->d.off, n + 1);
    std::vector<int32_t> o32;
    hipError_t e = d2h(o32, g->d.off, n + 1);
    off.assign(o32.begin(), o32.end());
    return e;
}

}  // namespace rs

using namespace rs;

// ================================================================== C ABI
// ------------------------------------------------------------ tiling
static rs_status check_tiling(const rs_tiling *t) {
    if (!t) return fail(RS_ERR_ARG, "tiling is NULL");
    if (t->row_entries < 64 || t->row_entries > kRowTile || t->row_vertices < 1 || t->row_vertices > kRowTileV ||
        t->score_pairs < 1 || t->score_pairs > kScoreTileP || t->score_vertices < 1 ||
        t->score_vertices > kScoreTileV || t->hub_list < 1 || t->hub_list > kHubList)
        return fail(RS_ERR_ARG, "tiling out of range: row_entries 64.." + std::to_string(kRowTile) +
                                    ", row_vertices 1.." + std::to_string(kRowTileV) + ", score_pairs 1.." +
                                    std::to_string(kScoreTileP) + ", score_vertices 1.." +
                                    std::to_string(kScoreTileV) + ", hub_list 1.." + std::to_string(kHubList));
    return RS_OK;
}

static Tiling to_tiling(const rs_tiling *t) {
    Tiling T;
    T.row_entries = t->row_entries;
    T.row_vertices = t->row_vertices;
    T.score_pairs = t->score_pairs;
    T.score_vertices = t->score_vertices;
    T.hub_list = t->hub_list;
    return T;
}

// A graph's schedule while a new one is made.
struct ScheduleState {
    DeviceGraph d;
    void *tile_slab, *gblk_slab;
    int n_rtiles, n_rhubs, n_stiles, n_shubs, n_schunks, n_schunks_lds, n_shubs_lds, grid_rows, grid_score;
    explicit ScheduleState(const rs_graph *g)
        : d(g->d), tile_slab(g->tile_slab), gblk_slab(g->gblk_slab), n_rtiles(g->n_rtiles), n_rhubs(g->n_rhubs),
          n_stiles(g->n_stiles), n_shubs(g->n_shubs), n_schunks(g->n_schunks), n_schunks_lds(g->n_schunks_lds),
          n_shubs_lds(g->n_shubs_lds), grid_rows(g->grid_rows), grid_score(g->grid_score) {}
    // The new one did not come about: free what there is of it, keep this one.
    void restore(rs_graph *g) const {
        if (g->tile_slab != tile_slab) dev_free(g, &g->tile_slab);
        if (g->gblk_slab != gblk_slab) dev_free(g, &g->gblk_slab);
        g->d = d;
        g->tile_slab = tile_slab;
        g->gblk_slab = gblk_slab;
        g->n_rtiles = n_rtiles;
        g->n_rhubs = n_rhubs;
        g->n_stiles = n_stiles;
        g->n_shubs = n_shubs;
        g->n_schunks = n_schunks;
        g->n_schunks_lds = n_schunks_lds;
        g->n_shubs_lds = n_shubs_lds;
        g->grid_rows = grid_rows;
        g->grid_score = grid_score;
    }
    // The new one is in place: free this one (the stream is idle).
    void drop(rs_graph *g) const {
        void *p = tile_slab;
        if (g->tile_slab != p) dev_free(g, &p);
        p = gblk_slab;
        if (g->gblk_slab != p) dev_free(g, &p);
    }
};

// Re-cut the schedule of a resident graph for the tiling T.  The cut needs
// each vertex's row capacity and load-time foreign degree, which the device
// keeps as the capacity layout and the pair-slot offsets; the tiles are cut
// on the host and the schedule's arrays replaced, and the graph must be scored
// again.  The old schedule goes once the new one is in place: on an error the
// graph keeps it, its tiling and its results.
static rs_status retile(rs_graph *g, const Tiling &T) {
    DeviceGraph &D = g->d;
    const int64_t n = D.n;
    hipError_t e = hipStreamSynchronize(g->stream);
    if (e != hipSuccess) return hip_fail(e, "retile");
    std::vector<int64_t> off, cap, fgn;
    std::vector<int32_t> goff;
    HostTiles X;
    try {
        off.resize(n + 1);
        goff.resize(n + 1);
        cap.resize(n);
        fgn.resize(n);
        if (D.off64) {
            e = hipMemcpy(off.data(), D.off, 8 * (size_t)(n + 1), hipMemcpyDeviceToHost);
        } else {
            std::vector<int32_t> o32(n + 1);
            e = hipMemcpy(o32.data(), D.off, 4 * (size_t)(n + 1), hipMemcpyDeviceToHost);
            for (int64_t v = 0; v <= n; ++v) off[v] = o32[v];
        }
        if (e == hipSuccess) e = hipMemcpy(goff.data(), D.goff, 4 * (size_t)(n + 1), hipMemcpyDeviceToHost);
        if (e != hipSuccess) return hip_fail(e, "retile: reading the capacity layout");
        for (int64_t v = 0; v < n; ++v) {
            cap[v] = off[v + 1] - off[v];
            fgn[v] = goff[v + 1] - goff[v];
        }
        cut_all(n, off, cap, fgn, g->h_vstart, T, X);
    } catch (const std::bad_alloc &) {
        return fail(RS_ERR_NOMEM, "host allocation failed while cutting tiles");
    }
    const ScheduleState old(g);
    rs_status st = upload_tiles(g, X);
    if (st == RS_OK && g->n_graphs > 0) {  // a batch's row blocks of each graph
        const DevReq reqs[] = {
            {(void **)&D.gblk_off, 4 * X.gblk_off.size()},
            {(void **)&D.gblk, 4 * std::max<size_t>(X.gblk.size(), 1)},
        };
        e = dev_alloc_group(g, reqs, 2, &g->gblk_slab);
        if (e == hipSuccess)
            e = hipMemcpyAsync(D.gblk_off, X.gblk_off.data(), 4 * X.gblk_off.size(), hipMemcpyHostToDevice, g->stream);
        if (e == hipSuccess && !X.gblk.empty())
            e = hipMemcpyAsync(D.gblk, X.gblk.data(), 4 * X.gblk.size(), hipMemcpyHostToDevice, g->stream);
        if (e != hipSuccess) st = hip_fail(e, "retile: batch row blocks");
    }
    e = hipStreamSynchronize(g->stream);  // (on an error too: the copies read this frame's arrays)
    if (st == RS_OK && e != hipSuccess) st = hip_fail(e, "retile");
    if (st != RS_OK) {
        (void)hipGetLastError();  // a failed allocation is not the next launch's error
        old.restore(g);
        return st;
    }
    old.drop(g);
    if (g->n_graphs > 0) {
        g->h_gblk_off.swap(X.gblk_off);
        g->h_gblk.swap(X.gblk);
    }
    g->tiling = T;
    g->scored = false;
    return st;
}

extern "C" {

const char *rs_status_string(rs_status s) {
    switch (s) {
        case RS_OK: return "RS_OK";
        case RS_ERR_ARG: return "RS_ERR_ARG";
        case RS_ERR_GRAPH: return "RS_ERR_GRAPH";
        case RS_ERR_RANGE: return "RS_ERR_RANGE";
        case RS_ERR_NOMEM: return "RS_ERR_NOMEM";
        case RS_ERR_HIP: return "RS_ERR_HIP";
        case RS_ERR_STATE: return "RS_ERR_STATE";
        default: return "RS_ERR_UNKNOWN";
    }
}

const char *rs_last_error(void) { return g_err.c_str(); }

// A batch passes its graph starts (n_graphs + 1 entries), else vstart is NULL.
static rs_status load_graph(const rs_csr *csr, void *hip_stream, uint32_t flags, const int64_t *vstart,
                            int32_t n_graphs, rs_graph **out) {
    if (!out) return fail(RS_ERR_ARG, "out is NULL");
    *out = nullptr;
    if (!csr) return fail(RS_ERR_ARG, "csr is NULL");
    if ((flags & ~RS_LOAD_WIDE_OFFSETS) != 0) return fail(RS_ERR_ARG, "unknown flags");
    if (csr->n < 0 || csr->nnz < 0) return fail(RS_ERR_ARG, "negative n or nnz");
    if (csr->offset_bytes != 4 && csr->offset_bytes != 8) return fail(RS_ERR_ARG, "offset_bytes must be 4 or 8");
    if (csr->on_device != 0 && csr->on_device != 1) return fail(RS_ERR_ARG, "on_device must be 0 or 1");
    if (!csr->row_offsets) return fail(RS_ERR_ARG, "row_offsets is NULL");
    if (csr->n > 0 && !csr->labels) return fail(RS_ERR_ARG, "labels is NULL");
    if (csr->nnz > 0 && !csr->col) return fail(RS_ERR_ARG, "col is NULL");
    if (csr->n > (int64_t)INT32_MAX - 1) return fail(RS_ERR_RANGE, "n does not fit int32 vertex ids");
    if (csr->offset_bytes == 4 && csr->nnz > (int64_t)INT32_MAX)
        return fail(RS_ERR_RANGE, "nnz overflows 4-byte row offsets");
    rs_graph *g = new (std::nothrow) rs_graph();
    if (!g) return fail(RS_ERR_NOMEM, "handle allocation failed");
    g->stream = (hipStream_t)hip_stream;  // NULL: created after validation
    g->wide_offsets = (flags & RS_LOAD_WIDE_OFFSETS) != 0;
    if (vstart) {
        g->n_graphs = n_graphs;
        g->h_vstart.assign(vstart, vstart + n_graphs + 1);
    }
    rs_status st = csr->offset_bytes == 8 ? load_t<int64_t>(csr, g) : load_t<int32_t>(csr, g);
    if (st != RS_OK) {
        std::string keep = g_err;
        release(g);
        delete g;
        g_err = keep;
        return st;
    }
    *out = g;
    return RS_OK;
}

rs_status rs_load_graph(const rs_csr *csr, void *hip_stream, uint32_t flags, rs_graph **out) {
    clear_error();
    return load_graph(csr, hip_stream, flags, nullptr, 0, out);
}

// Bytes of a batch's top-k block: counts, scores, ids.
static size_t batch_out_bytes(size_t graphs, size_t k) { return 8 * graphs + 12 * graphs * k; }

rs_status rs_load_batch(int32_t n_graphs, const int64_t *vertex_offsets, const rs_csr *csr, void *hip_stream,
                        uint32_t flags, rs_graph **out) {
    clear_error();
    if (!out) return fail(RS_ERR_ARG, "out is NULL");
    *out = nullptr;
    if (n_graphs < 1 || !vertex_offsets || !csr) return fail(RS_ERR_ARG, "n_graphs < 1, or a NULL array");
    if (csr->on_device) return fail(RS_ERR_ARG, "a batch is loaded from host arrays");
    if (csr->n < 0 || csr->nnz < 0) return fail(RS_ERR_ARG, "negative n or nnz");
    if (csr->offset_bytes != 4 && csr->offset_bytes != 8) return fail(RS_ERR_ARG, "offset_bytes must be 4 or 8");
    if (!csr->row_offsets || (csr->n > 0 && !csr->labels) || (csr->nnz > 0 && !csr->col))
        return fail(RS_ERR_ARG, "null CSR array");
    const int64_t n = csr->n;
    if (vertex_offsets[0] != 0 || vertex_offsets[n_graphs] != n) return fail(RS_ERR_ARG, "vertex_offsets must run 0..n");
    for (int32_t gi = 0; gi < n_graphs; ++gi)
        if (vertex_offsets[gi + 1] < vertex_offsets[gi]) return fail(RS_ERR_ARG, "vertex_offsets decrease");
    auto rowoff = [&](int64_t v) {
        return csr->offset_bytes == 8 ? ((const int64_t *)csr->row_offsets)[v]
                                      : (int64_t)((const int32_t *)csr->row_offsets)[v];
    };
    // the row offsets first: the scan below walks every row
    if (rowoff(0) != 0) return fail(RS_ERR_GRAPH, "row_offsets[0] != 0");
    for (int64_t v = 0; v < n; ++v)
        if (rowoff(v + 1) < rowoff(v)) return fail(RS_ERR_GRAPH, "row_offsets decrease at vertex " + std::to_string(v));
    if (rowoff(n) != csr->nnz) return fail(RS_ERR_GRAPH, "row_offsets[n] != nnz");
    // every edge stays inside its graph; labels are ranked per graph and
    // offset so that no community spans two graphs (the ranks keep each
    // graph's label order, hence its internal numbering)
    std::vector<int32_t> lab2;
    try {
        lab2.resize(n);
        int64_t base = 0;
        for (int32_t gi = 0; gi < n_graphs; ++gi) {
            const int64_t a = vertex_offsets[gi], b = vertex_offsets[gi + 1];
            for (int64_t v = a; v < b; ++v)
                for (int64_t e = rowoff(v); e < rowoff(v + 1); ++e)
                    if (csr->col[e] < a || csr->col[e] >= b) return fail(RS_ERR_GRAPH, "an edge joins two graphs of the batch");
            std::vector<int32_t> u(csr->labels + a, csr->labels + b);
            std::sort(u.begin(), u.end());
            u.erase(std::unique(u.begin(), u.end()), u.end());
            for (int64_t v = a; v < b; ++v) {
                if (csr->labels[v] < 0) return fail(RS_ERR_GRAPH, "negative label");
                lab2[v] = (int32_t)(base + (std::lower_bound(u.begin(), u.end(), csr->labels[v]) - u.begin()));
            }
            base += (int64_t)u.size();
            if (base > (int64_t)INT32_MAX) return fail(RS_ERR_RANGE, "too many communities in the batch");
        }
    } catch (const std::bad_alloc &) {
        return fail(RS_ERR_NOMEM, "host staging of the batch failed");
    }
    rs_csr c = *csr;
    c.labels = lab2.data();
    rs_graph *g = nullptr;
    rs_status st = load_graph(&c, hip_stream, flags, vertex_offsets, n_graphs, &g);
    if (st != RS_OK) return st;
    DeviceGraph &D = g->d;
    std::vector<int32_t> vg(n);
    for (int32_t gi = 0; gi < n_graphs; ++gi)
        for (int64_t v = vertex_offsets[gi]; v < vertex_offsets[gi + 1]; ++v) vg[v] = gi;
    const size_t N = (size_t)std::max<int64_t>(n, 1), G = (size_t)n_graphs;
    const DevReq reqs[] = {
        {(void **)&D.vstart, 8 * (G + 1)},
        {(void **)&D.vgraph, 4 * N},
        {(void **)&D.gwmax, 8 * G},
        {(void **)&D.gorder, 4 * G},
        {(void **)&D.bout, batch_out_bytes(G, kBatchK)},
    };
    hipError_t e = dev_alloc_group(g, reqs, sizeof(reqs) / sizeof(reqs[0]));
    // (replaced when the schedule is cut again)
    const DevReq blocks[] = {
        {(void **)&D.gblk_off, 4 * (G + 1)},
        {(void **)&D.gblk, 4 * std::max<size_t>(g->h_gblk.size(), 1)},
    };
    if (e == hipSuccess) e = dev_alloc_group(g, blocks, 2, &g->gblk_slab);
    if (e == hipSuccess) e = hipMemcpyAsync(D.vstart, vertex_offsets, 8 * (G + 1), hipMemcpyHostToDevice, g->stream);
    if (e == hipSuccess && n) e = hipMemcpyAsync(D.vgraph, vg.data(), 4 * n, hipMemcpyHostToDevice, g->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(D.gblk_off, g->h_gblk_off.data(), 4 * (G + 1), hipMemcpyHostToDevice, g->stream);
    // top-k segments, when every graph has at most kSegMax of them
    int64_t nmax = 0;
    for (size_t i = 0; i < G; ++i) nmax = std::max<int64_t>(nmax, vertex_offsets[i + 1] - vertex_offsets[i]);
    std::vector<int32_t> seg_g, sfirst(G + 1, 0);
    if (nmax <= (int64_t)kSegVerts * kSegMax) {
        for (size_t i = 0; i < G; ++i) {
            const int64_t ns = (vertex_offsets[i + 1] - vertex_offsets[i] + kSegVerts - 1) / kSegVerts;
            for (int64_t j = 0; j < ns; ++j) seg_g.push_back((int32_t)i);
            sfirst[i + 1] = (int32_t)seg_g.size();
            if (ns > 0) ++g->n_graphs_seg;
        }
    }
    const size_t S = seg_g.size();
    if (e == hipSuccess && S > 0) {
        const DevReq more[] = {
            {(void **)&D.seg_g, 4 * S},
            {(void **)&D.sfirst, 4 * (G + 1)},
            {(void **)&D.c_hi, 8 * S * kBatchK},
            {(void **)&D.c_lo, 4 * S * kBatchK},
            {(void **)&D.c_cnt, 4 * S},
        };
        e = dev_alloc_group(g, more, sizeof(more) / sizeof(more[0]));
        if (e == hipSuccess) e = hipMemcpyAsync(D.seg_g, seg_g.data(), 4 * S, hipMemcpyHostToDevice, g->stream);
        if (e == hipSuccess) e = hipMemcpyAsync(D.sfirst, sfirst.data(), 4 * (G + 1), hipMemcpyHostToDevice, g->stream);
        if (e == hipSuccess) g->n_segs = (int32_t)S;
    }
    std::vector<int32_t> order(G);
    for (size_t i = 0; i < G; ++i) order[i] = (int32_t)i;
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
        return vertex_offsets[a + 1] - vertex_offsets[a] > vertex_offsets[b + 1] - vertex_offsets[b];
    });
    if (e == hipSuccess) e = hipMemcpyAsync(D.gorder, order.data(), 4 * G, hipMemcpyHostToDevice, g->stream);
    if (e == hipSuccess && !g->h_gblk.empty())
        e = hipMemcpyAsync(D.gblk, g->h_gblk.data(), 4 * g->h_gblk.size(), hipMemcpyHostToDevice, g->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(g->stream);
    if (e != hipSuccess) {
        st = hip_fail(e, "batch upload");
        std::string keep = g_err;
        rs_free_graph(g);
        g_err = keep;
        return st;
    }
    *out = g;
    return RS_OK;
}

rs_status rs_topk_batch(rs_graph *g, int64_t k, int32_t *ids, double *scores, int64_t *counts) {
    clear_error();
    if (!g || !ids || !scores || !counts) return fail(RS_ERR_ARG, "graph or an output is NULL");
    if (g->n_graphs <= 0) return fail(RS_ERR_STATE, "not a batch");
    if (k < 1 || k > kBatchK) return fail(RS_ERR_ARG, "k must be 1.." + std::to_string(kBatchK));
    if (!g->scored) return fail(RS_ERR_STATE, "rs_topk_batch before rs_score");
    const size_t G = (size_t)g->n_graphs, bytes = batch_out_bytes(G, (size_t)k);
    if (!g->bpin) {
        const hipError_t ea = hipHostMalloc((void **)&g->bpin, batch_out_bytes(G, kBatchK), hipHostMallocDefault);
        if (ea != hipSuccess) {
            g->bpin = nullptr;
            return hip_fail(ea, "pinned batched top-k buffer");
        }
    }
    // one block and one copy: counts, scores, ids
    char *o = g->d.bout;
    const size_t o_sc = 8 * G, o_id = o_sc + 8 * G * (size_t)k;
    rs_status st = launch_topk_graphs(g, k, (int32_t *)(o + o_id), (double *)(o + o_sc), (int64_t *)o);
    if (st != RS_OK) return st;
    hipError_t e = hipMemcpyAsync(g->bpin, o, bytes, hipMemcpyDeviceToHost, g->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(g->stream);
    if (e != hipSuccess) return hip_fail(e, "batched top-k copy");
    memcpy(counts, g->bpin, 8 * G);
    memcpy(scores, g->bpin + o_sc, 8 * G * (size_t)k);
    memcpy(ids, g->bpin + o_id, 4 * G * (size_t)k);
    for (size_t i = 0; i < G; ++i)  // a graph with fewer live vertices than k
        for (int64_t j = counts[i]; j < k; ++j) {
            ids[i * (size_t)k + j] = 0;
            scores[i * (size_t)k + j] = 0.0;
        }
    return RS_OK;
}

void rs_free_graph(rs_graph *g) {
    if (!g) return;
    if (g->stream) (void)hipStreamSynchronize(g->stream);
    release(g);
    delete g;
}

rs_status rs_score(rs_graph *g) {
    clear_error();
    if (!g) return fail(RS_ERR_ARG, "graph is NULL");
    rs_status st = launch_score_pass(g);
    if (st == RS_OK) g->scored = true;
    return st;
}

rs_status rs_topk(rs_graph *g, int64_t k, int32_t *ids, double *scores, int64_t *count) {
    clear_error();
    if (!g || !count) return fail(RS_ERR_ARG, "graph or count is NULL");
    if (k < 0) return fail(RS_ERR_ARG, "k < 0");
    if (k > 0 && (!ids || !scores)) return fail(RS_ERR_ARG, "ids or scores is NULL");
    if (!g->scored) return fail(RS_ERR_STATE, "rs_topk before rs_score");
    int64_t cnt = 0;
    rs_status st = launch_topk(g, k, ids, scores, &cnt);
    if (st != RS_OK) return st;
    *count = cnt;
    return RS_OK;
}

// Batches of up to this many ids are read from pinned memory by the removal
// kernel itself: a copy before it costs 3 to 6 us (a
// request of 200 edges and 5 vertices at n = 1 million: 185 against 190 us).
constexpr int64_t kDirectIds = 8192;
// The edges of up to this many are looked up among the listed vertices, to
// remove both in one launch (two launches: 13 us more).
constexpr int64_t kApartMax = 16384;

rs_status rs_apply_removals(rs_graph *g, const rs_removals *b, rs_removal_result *res) {
    clear_error();
    if (!g || !b) return fail(RS_ERR_ARG, "graph or batch is NULL");
    if (!g->scored) return fail(RS_ERR_STATE, "rs_apply_removals before rs_score");
    if (g->n_graphs > 0) return fail(RS_ERR_STATE, "removals are not applied to a batch of graphs");
    if (b->n_edges < 0 || b->n_vertices < 0) return fail(RS_ERR_ARG, "negative batch size");
    if (b->n_edges > 0 && (!b->src || !b->dst)) return fail(RS_ERR_ARG, "edge arrays are NULL");
    if (b->n_vertices > 0 && !b->vertices) return fail(RS_ERR_ARG, "vertex array is NULL");
    const int64_t n = g->d.n;
    std::vector<int32_t> es, ed, vs;
    try {
        es.resize(b->n_edges);
        ed.resize(b->n_edges);
        vs.resize(b->n_vertices);
    } catch (const std::bad_alloc &) {
        return fail(RS_ERR_NOMEM, "host staging allocation failed");
    }
    for (int64_t i = 0; i < b->n_edges; ++i) {
        const int32_t a = b->src[i], c = b->dst[i];
        if (a < 0 || a >= n || c < 0 || c >= n) return fail(RS_ERR_RANGE, "edge endpoint out of range");
        es[i] = g->h_old2new[a];
        ed[i] = g->h_old2new[c];
    }
    for (int64_t i = 0; i < b->n_vertices; ++i) {
        const int32_t x = b->vertices[i];
        if (x < 0 || x >= n) return fail(RS_ERR_RANGE, "vertex id out of range");
        vs[i] = g->h_old2new[x];
    }
    std::sort(vs.begin(), vs.end());
    vs.erase(std::unique(vs.begin(), vs.end()), vs.end());
    const int64_t m = b->n_edges, nv = (int64_t)vs.size();
    bool apart = m == 0 || nv == 0 || m <= kApartMax;  // no listed edge has a listed vertex
    for (int64_t i = 0; nv > 0 && apart && i < m; ++i)
        apart = !std::binary_search(vs.begin(), vs.end(), es[i]) && !std::binary_search(vs.begin(), vs.end(), ed[i]);
    const int64_t need = std::max<int64_t>(2 * m + nv, 1);
    // staging kept between calls: grown (never shrunk) before anything is mutated
    if (need > g->rem_cap || need > g->rem_host_cap) {
        const int64_t cap = std::max<int64_t>(2 * need, 4096);
        int32_t *nb = nullptr, *nh = nullptr;
        hipError_t ea = hipMalloc((void **)&nb, 4 * (size_t)cap);
        if (ea == hipSuccess) ea = hipHostMalloc((void **)&nh, 4 * (size_t)cap, hipHostMallocDefault);
        if (ea != hipSuccess) {
            if (nb) (void)hipFree(nb);
            return hip_fail(ea, "removal staging");
        }
        if (g->rem_buf) (void)hipFree(g->rem_buf);
        if (g->rem_host) (void)hipHostFree(g->rem_host);
        g->dev_bytes += 4 * (cap - g->rem_cap);  // the device staging counts toward the graph's footprint
        g->rem_buf = nb;
        g->rem_host = nh;
        g->rem_cap = g->rem_host_cap = cap;
    }
    std::copy(es.begin(), es.end(), g->rem_host);
    std::copy(ed.begin(), ed.end(), g->rem_host + m);
    std::copy(vs.begin(), vs.end(), g->rem_host + 2 * m);
    const int32_t *buf = g->rem_host;
    hipError_t e = hipSuccess;
    if (need > kDirectIds) {
        e = hipMemcpyAsync(g->rem_buf, g->rem_host, 4 * (size_t)(2 * m + nv), hipMemcpyHostToDevice, g->stream);
        buf = g->rem_buf;
    }
    if (e == hipSuccess && g->ictr_dirty) {
        e = hipMemsetAsync(g->d.ictr, 0, 8 * (size_t)kIcCount, g->stream);
        if (e == hipSuccess) e = hipMemsetAsync(g->d.ictr_next, 0, 8 * (size_t)kIcCount, g->stream);
    }
    rs_status st = e == hipSuccess ? RS_OK : hip_fail(e, "removal upload");
    // remove (marking the rows that change), then compact those rows, find
    // what must be recomputed and rerun only that; a listed edge at a listed
    // vertex is the edge's to remove, so then the edges go first
    g->ictr_dirty = true;
    *g->rem_cnt_host = RemovalCounts{0, 0, 0, 0};
    if (st == RS_OK && apart) {
        st = launch_remove(g, buf, buf + m, m, buf + 2 * m, nv);
    } else if (st == RS_OK) {
        st = launch_remove(g, buf, buf + m, m, nullptr, 0);
        if (st == RS_OK) st = launch_remove(g, nullptr, nullptr, 0, buf + 2 * m, nv);
    }
    // The marks leave the counts in pinned memory, behind an event, and the
    // pass (sized on the device) is queued right after it: the host waits for
    // the counts while the GPU goes on.
    if (st == RS_OK) st = launch_incremental_marks(g);
    if (st == RS_OK) {
        e = hipEventRecord(g->rem_ev, g->stream);
        if (e != hipSuccess) st = hip_fail(e, "incremental counts");
    }
    if (st == RS_OK) st = launch_score_incremental(g);
    if (st == RS_OK) {
        e = hipEventSynchronize(g->rem_ev);
        if (e != hipSuccess) st = hip_fail(e, "incremental counts");
    }
    // the re-score stays queued on the graph's stream (as rs_score's pass)
    if (st != RS_OK) {
        (void)hipStreamSynchronize(g->stream);  // what was queued reads the staging
        return st;
    }
    g->ictr_dirty = false;
    std::swap(g->d.ictr, g->d.ictr_next);  // (the marks have cleared the next one's)
    const RemovalCounts c = *g->rem_cnt_host;
    g->n_alive -= (int64_t)c.vertices;
    if (res) {
        res->edges_removed = (int64_t)(c.edges + c.vertex_edges);
        res->edges_ignored = m - (int64_t)c.edges;
        res->vertices_removed = (int64_t)c.vertices;
        res->affected = (int64_t)c.affected;
    }
    return RS_OK;
}

rs_status rs_restrict_to_targets(rs_graph *g, int32_t k_c, rs_removal_result *res) {
    clear_error();
    if (!g) return fail(RS_ERR_ARG, "graph is NULL");
    if (k_c < 1) return fail(RS_ERR_ARG, "k_c < 1");
    if (g->n_graphs > 0) return fail(RS_ERR_STATE, "target mode is not applied to a batch of graphs");
    // internal communities are numbered in ascending caller label, so a
    // stable sort by decreasing size breaks ties by the smaller label
    const int64_t k = g->d.k;
    std::vector<int32_t> cs, order, drop;
    hipError_t e = d2h(cs, g->d.cstart, k + 1);
    if (e != hipSuccess) return hip_fail(e, "community ranges");
    try {
        order.resize(k);
        for (int64_t c = 0; c < k; ++c) order[c] = (int32_t)c;
        std::stable_sort(order.begin(), order.end(),
                         [&](int32_t a, int32_t b) { return cs[a + 1] - cs[a] > cs[b + 1] - cs[b]; });
        for (int64_t i = k_c; i < k; ++i)
            for (int32_t v = cs[order[i]]; v < cs[order[i] + 1]; ++v) drop.push_back(g->h_new2old[v]);
    } catch (const std::bad_alloc &) {
        return fail(RS_ERR_NOMEM, "host staging allocation failed");
    }
    if (!g->scored) {
        rs_status st = launch_score_pass(g);
        if (st != RS_OK) return st;
        g->scored = true;
    }
    if (drop.empty()) {
        if (res) *res = rs_removal_result{0, 0, 0, 0};
        return RS_OK;
    }
    rs_removals b{0, nullptr, nullptr, (int64_t)drop.size(), drop.data()};
    return rs_apply_removals(g, &b, res);
}

rs_status rs_reachable_communities(rs_graph *g, int64_t n_sources, const int32_t *sources, int64_t *counts) {
    clear_error();
    if (!g) return fail(RS_ERR_ARG, "graph is NULL");
    if (n_sources < 0 || n_sources > kMaxReachSources)
        return fail(RS_ERR_ARG, "n_sources must be 0.." + std::to_string(kMaxReachSources));
    if (n_sources > 0 && (!sources || !counts)) return fail(RS_ERR_ARG, "sources or counts is NULL");
    const int64_t n = g->d.n;
    for (int64_t i = 0; i < n_sources; ++i)
        if (sources[i] < 0 || sources[i] >= n) return fail(RS_ERR_RANGE, "source id out of range");
    if (n_sources == 0) return RS_OK;
    const int words = std::max(1, (int)((g->d.k + 31) / 32));
    // buffers kept by the handle from the first call (sized for the largest
    // source count, 1,024)
    hipError_t e = hipSuccess;
    const size_t cap = 12 * (size_t)kMaxReachSources;  // counts and sources
    if (!g->reach_comp) {
        e = dev_alloc(g, (void **)&g->reach_comp, 4 * (size_t)std::max<int64_t>(n, 1));
        if (e == hipSuccess) e = dev_alloc(g, (void **)&g->reach_bits, 4 * (size_t)kMaxReachSources * words);
        if (e == hipSuccess) e = dev_alloc(g, (void **)&g->reach_cnt, cap);
        if (e == hipSuccess && !g->reach_host) e = hipHostMalloc((void **)&g->reach_host, cap, hipHostMallocDefault);
        if (e != hipSuccess) {
            g->reach_comp = nullptr;  // (device buffers stay tracked and are freed with the handle)
            return hip_fail(e, "reach buffers");
        }
    }
    int32_t *src = (int32_t *)(g->reach_host + kMaxReachSources);
    int32_t *d_src = (int32_t *)(g->reach_cnt + kMaxReachSources);
    for (int64_t i = 0; i < n_sources; ++i) src[i] = g->h_old2new[sources[i]];
    e = hipMemcpyAsync(d_src, src, 4 * (size_t)n_sources, hipMemcpyHostToDevice, g->stream);
    rs_status st = e == hipSuccess ? RS_OK : hip_fail(e, "reach upload");
    if (st == RS_OK) st = launch_reach(g, d_src, (int)n_sources, g->reach_comp, g->reach_bits, words, g->reach_cnt);
    if (st == RS_OK) {
        e = hipMemcpyAsync(g->reach_host, g->reach_cnt, 8 * (size_t)n_sources, hipMemcpyDeviceToHost, g->stream);
        if (e != hipSuccess) st = hip_fail(e, "reach copy");
    }
    e = hipStreamSynchronize(g->stream);  // (on an error too: the upload reads the pinned sources)
    if (st == RS_OK && e != hipSuccess) st = hip_fail(e, "reach copy");
    if (st == RS_OK)
        for (int64_t i = 0; i < n_sources; ++i) counts[i] = g->reach_host[i];
    return st;
}

// Scratch layout of rs_reachable_communities_static (offsets from the
// device's static array, each 256-byte aligned): the counts, the sources, the
// community bitmaps, the component labels.
static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

rs_status rs_reachable_communities_static(rs_graph *g, int64_t n_sources, const int32_t *sources, int64_t *counts) {
    clear_error();
    if (!g) return fail(RS_ERR_ARG, "graph is NULL");
    if (n_sources < 0 || n_sources > kMaxReachSources)
        return fail(RS_ERR_ARG, "n_sources must be 0.." + std::to_string(kMaxReachSources));
    if (n_sources > 0 && (!sources || !counts)) return fail(RS_ERR_ARG, "sources or counts is NULL");
    const int64_t n = g->d.n;
    int32_t src[kMaxReachSources];
    for (int64_t i = 0; i < n_sources; ++i) {
        if (sources[i] < 0 || sources[i] >= n) return fail(RS_ERR_RANGE, "source id out of range");
        src[i] = g->h_old2new[sources[i]];
    }
    if (n_sources == 0) return RS_OK;
    const int words = std::max(1, (int)((g->d.k + 31) / 32));
    const size_t o_cnt = 256, o_src = o_cnt + align256(8 * (size_t)n_sources),
                 o_bits = o_src + align256(4 * (size_t)n_sources),
                 o_comp = o_bits + align256(4 * (size_t)n_sources * words),
                 need = o_comp + 4 * (size_t)std::max<int64_t>(n, 1);
    if (need > kStaticScratchBytes)
        return fail(RS_ERR_RANGE, "graph too large for the static scratch: needs " + std::to_string(need) +
                                      " bytes (4 per vertex plus the bitmaps), at most " +
                                      std::to_string(kStaticScratchBytes));
    void *base = nullptr;
    rs_status st = static_scratch(g->device, &base);
    if (st != RS_OK) return st;
    char *b = (char *)base;
    long long *d_cnt = (long long *)(b + o_cnt);
    int32_t *d_src = (int32_t *)(b + o_src);
    unsigned int *d_bits = (unsigned int *)(b + o_bits);
    int32_t *d_comp = (int32_t *)(b + o_comp);
    hipError_t e = hipMemcpyAsync(d_src, src, 4 * (size_t)n_sources, hipMemcpyHostToDevice, g->stream);
    if (e != hipSuccess) return hip_fail(e, "reach upload");
    st = launch_reach(g, d_src, (int)n_sources, d_comp, d_bits, words, d_cnt);
    if (st == RS_OK) {
        e = hipMemcpyAsync(counts, d_cnt, 8 * (size_t)n_sources, hipMemcpyDeviceToHost, g->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(g->stream);
        if (e != hipSuccess) st = hip_fail(e, "reach copy");
    } else {
        (void)hipStreamSynchronize(g->stream);  // the source upload reads this frame's array
    }
    return st;
}

rs_status rs_get_tiling(rs_graph *g, rs_tiling *t) {
    clear_error();
    if (!g || !t) return fail(RS_ERR_ARG, "graph or tiling is NULL");
    t->row_entries = g->tiling.row_entries;
    t->row_vertices = g->tiling.row_vertices;
    t->score_pairs = g->tiling.score_pairs;
    t->score_vertices = g->tiling.score_vertices;
    t->hub_list = g->tiling.hub_list;
    return RS_OK;
}

rs_status rs_set_tiling(rs_graph *g, const rs_tiling *t) {
    clear_error();
    if (!g) return fail(RS_ERR_ARG, "graph is NULL");
    rs_status st = check_tiling(t);
    if (st != RS_OK) return st;
    return retile(g, to_tiling(t));
}

rs_status rs_autotune(rs_graph *g, int32_t n_cand, const rs_tiling *cand, int32_t reps, int32_t *best, double *ms) {
    clear_error();
    if (!g || !cand || !best || !ms) return fail(RS_ERR_ARG, "graph, candidates, best or ms is NULL");
    if (n_cand < 1 || reps < 1) return fail(RS_ERR_ARG, "n_cand and reps must be >= 1");
    for (int32_t i = 0; i < n_cand; ++i) {
        const rs_status st = check_tiling(&cand[i]);
        if (st != RS_OK) return st;
    }
    const bool was_scored = g->scored;
    const Tiling before = g->tiling;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    rs_status st = e == hipSuccess ? RS_OK : hip_fail(e, "autotune events");
    int32_t b = -1;
    for (int32_t i = 0; i < n_cand && st == RS_OK; ++i) {
        st = retile(g, to_tiling(&cand[i]));
        if (st == RS_OK) st = launch_score_pass(g);  // warm-up
        if (st != RS_OK) break;
        e = hipEventRecord(e0, g->stream);
        for (int32_t r = 0; r < reps && st == RS_OK && e == hipSuccess; ++r) st = launch_score_pass(g);
        if (e == hipSuccess) e = hipEventRecord(e1, g->stream);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        float t = 0.f;
        if (e == hipSuccess) e = hipEventElapsedTime(&t, e0, e1);
        if (e != hipSuccess && st == RS_OK) st = hip_fail(e, "autotune timing");
        ms[i] = (double)t / reps;
        if (st == RS_OK && (b < 0 || ms[i] < ms[b])) b = i;
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (st == RS_OK) st = retile(g, to_tiling(&cand[b]));
    if (st == RS_OK) {
        *best = b;
    } else if (b >= 0) {  // back to the cut-offs before the first candidate
        std::string keep = g_err;
        if (retile(g, before) != RS_OK) return st;  // (g holds a candidate's, to be scored)
        g_err = keep;
    }
    if (was_scored && !g->scored) {
        const rs_status ss = launch_score_pass(g);
        if (ss == RS_OK) g->scored = true;
        if (st == RS_OK) st = ss;
    }
    return st;
}

rs_status rs_read_scores(rs_graph *g, double *out, int64_t n, int32_t raw) {
    clear_error();
    if (!g || (!out && n > 0)) return fail(RS_ERR_ARG, "graph or out is NULL");
    if (n != g->d.n) return fail(RS_ERR_ARG, "n does not match the graph");
    if (!g->scored) return fail(RS_ERR_STATE, "rs_read_scores before rs_score");
    if (n == 0) return RS_OK;
    rs_status st = launch_gather_scores(g, g->d.scratch_d, raw ? 1 : 0);
    if (st != RS_OK) return st;
    return fetch(g, {{out, g->d.scratch_d, 8 * (size_t)n}}, "score copy");
}

rs_status rs_read_counts(rs_graph *g, rs_counts *c) {
    clear_error();
    if (!g || !c) return fail(RS_ERR_ARG, "graph or counts is NULL");
    if (g->scored) {
        const rs_status st = launch_reduce_counts(g);
        if (st != RS_OK) return st;
    }
    DevCounters dc;
    hipError_t e = hipMemcpyAsync(&dc, g->d.ctr, sizeof(dc), hipMemcpyDeviceToHost, g->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(g->stream);
    if (e != hipSuccess) return hip_fail(e, "counter copy");
    std::vector<int32_t> deg(g->d.n);
    if (g->d.n) {
        e = hipMemcpy(deg.data(), g->d.deg, 4 * g->d.n, hipMemcpyDeviceToHost);
        if (e != hipSuccess) return hip_fail(e, "degree copy");
    }
    int64_t live = 0;
    for (int32_t d : deg) live += d;
    c->n = g->d.n;
    c->nnz = live;
    c->n_alive = g->n_alive;
    c->n_communities = g->d.k;
    c->n_border = (int64_t)dc.n_border;
    c->m_inter = (int64_t)dc.sum_dprime / 2;
    c->sum_ell = (int64_t)dc.sum_ell;
    c->sum_ell_x = (int64_t)dc.sum_ell_x;
    c->sum_tI = (int64_t)dc.sum_tI;
    c->sum_tII = (int64_t)dc.sum_tII;
    c->sum_work_I = (int64_t)dc.sum_workI;
    double w;
    std::memcpy(&w, &dc.wmax_bits, sizeof(w));
    c->omega_max = w;
    return RS_OK;
}

rs_status rs_read_vertex_counts(rs_graph *g, int32_t *border, int32_t *ell, int32_t *dprime, int64_t *tI,
                                int64_t *tII, double *w_own) {
    clear_error();
    if (!g) return fail(RS_ERR_ARG, "graph is NULL");
    if (!g->scored) return fail(RS_ERR_STATE, "read before rs_score");
    const size_t n = (size_t)g->d.n;
    if (n == 0) return RS_OK;
    // gathered into the top-k's lists (16 bytes a vertex each), which hold
    // nothing between calls
    char *a = (char *)g->d.tfinal, *b = (char *)g->d.ttie, *c = (char *)g->d.ttie2;
    VertexOut o = {};
    if (tI) o.tI = (long long *)a;
    if (tII) o.tII = (long long *)(a + 8 * n);
    if (w_own) o.w_own = (double *)b;
    if (border) o.border = (int32_t *)(b + 8 * n);
    if (ell) o.ell = (int32_t *)(b + 12 * n);
    if (dprime) o.dprime = (int32_t *)c;
    const rs_status st = launch_gather_counts(g, o);
    if (st != RS_OK) return st;
    return fetch(g, {{tI, o.tI, 8 * n}, {tII, o.tII, 8 * n}, {w_own, o.w_own, 8 * n}, {border, o.border, 4 * n},
                     {ell, o.ell, 4 * n}, {dprime, o.dprime, 4 * n}}, "vertex count copy");
}

rs_status rs_read_rows(rs_graph *g, int64_t *row_off, int32_t *comm, int32_t *count, double *weight) {
    clear_error();
    if (!g || !row_off) return fail(RS_ERR_ARG, "graph or row_off is NULL");
    if (!g->scored) return fail(RS_ERR_STATE, "read before rs_score");
    const int64_t n = g->d.n;
    hipError_t e = hipStreamSynchronize(g->stream);
    std::vector<VMeta> meta;
    if (e == hipSuccess) e = read_meta(g, meta);
    if (e != hipSuccess) return hip_fail(e, "row copy");
    row_off[0] = 0;
    for (int64_t v = 0; v < n; ++v) row_off[v + 1] = row_off[v] + meta[g->h_old2new[v]].ell;
    if (!comm && !count && !weight) return RS_OK;
    // a row's foreign records sit at the leader slots (a run's length leads
    // to the next leader); the own community's goes in by its number
    std::vector<int32_t> goff, lab;
    std::vector<PairRec> rec;
    std::vector<double> own;
    e = d2h(goff, g->d.goff, n + 1);
    if (e == hipSuccess) e = d2h(lab, g->d.lab, n);
    if (e == hipSuccess) e = d2h(own, g->d.wown, n);
    if (e == hipSuccess) e = d2h(rec, g->d.prec, n ? goff[n] : 0);
    if (e != hipSuccess) return hip_fail(e, "row copy");
    for (int64_t v = 0; v < n; ++v) {
        const int32_t x = g->h_old2new[v];
        const VMeta &m = meta[x];
        int64_t o = row_off[v];
        auto put = [&](int32_t c, int32_t f, double w) {
            if (comm) comm[o] = g->h_comm2orig[c];
            if (count) count[o] = f;
            if (weight) weight[o] = w;
            ++o;
        };
        bool own_due = m.q > m.p;
        const int32_t s1 = goff[x] + m.deg - (m.q - m.p);
        for (int32_t s = goff[x]; s < s1; s += rec[s].f) {
            if (own_due && rec[s].c > lab[x]) {
                put(lab[x], m.q - m.p, own[x]);
                own_due = false;
            }
            put(rec[s].c, rec[s].f, rec[s].w);
        }
        if (own_due) put(lab[x], m.q - m.p, own[x]);
    }
    return RS_OK;
}

rs_status rs_read_gprime(rs_graph *g, int64_t *goff, int32_t *gcol) {
    clear_error();
    if (!g || !goff) return fail(RS_ERR_ARG, "graph or off is NULL");
    if (!g->scored) return fail(RS_ERR_STATE, "read before rs_score");
    const int64_t n = g->d.n;
    hipError_t e = hipStreamSynchronize(g->stream);
    std::vector<VMeta> meta;
    std::vector<int32_t> hcol;
    std::vector<int64_t> off;
    if (e == hipSuccess) e = read_meta(g, meta);
    if (e == hipSuccess) e = read_offsets(g, off);
    if (e != hipSuccess) return hip_fail(e, "G' copy");
    goff[0] = 0;
    for (int64_t v = 0; v < n; ++v) {
        const VMeta &m = meta[g->h_old2new[v]];
        goff[v + 1] = goff[v] + m.deg - (m.q - m.p);
    }
    if (!gcol) return RS_OK;
    e = d2h(hcol, g->d.col, g->d.nnz);
    if (e != hipSuccess) return hip_fail(e, "G' copy");
    for (int64_t v = 0; v < n; ++v) {
        const int32_t x = g->h_old2new[v];
        const VMeta &m = meta[x];
        const int64_t rb = off[x];
        int64_t o = goff[v];
        for (int32_t j = 0; j < m.deg; ++j) {
            if (j >= m.p && j < m.q) continue;
            gcol[o++] = g->h_new2old[hcol[rb + j]];
        }
        std::sort(gcol + goff[v], gcol + goff[v + 1]);
    }
    return RS_OK;
}

static const char *kKernelNames[K_COUNT] = {
    "k_rows", "k_mid", "k_score", "k_topk_hist", "k_topk_find", "k_topk_collect", "k_tie_rank", "k_final_order",
    "k_hub_sum", "k_topk_graphs"};

const char *rs_kernel_name(int32_t id) { return (id >= 0 && id < K_COUNT) ? kKernelNames[id] : nullptr; }

rs_status rs_set_timing(rs_graph *g, int32_t on) {
    clear_error();
    if (!g) return fail(RS_ERR_ARG, "graph is NULL");
    g->timing.on = on != 0;
    return RS_OK;
}

rs_status rs_read_timings(rs_graph *g, int32_t cap, double *ms, int64_t *launches, int32_t *n_kernels) {
    clear_error();
    if (!g) return fail(RS_ERR_ARG, "graph is NULL");
    hipError_t e = hipStreamSynchronize(g->stream);
    if (e != hipSuccess) return hip_fail(e, "timing sync");
    for (auto &pe : g->timing.pending) {
        float t = 0.f;
        if (hipEventElapsedTime(&t, pe.second.first, pe.second.second) == hipSuccess) {
            g->timing.ms[pe.first] += t;
            g->timing.launches[pe.first] += 1;
        }
        g->timing.pool.push_back(pe.second.first);
        g->timing.pool.push_back(pe.second.second);
    }
    g->timing.pending.clear();
    for (int i = 0; i < K_COUNT && i < cap; ++i) {
        if (ms) ms[i] = g->timing.ms[i];
        if (launches) launches[i] = g->timing.launches[i];
    }
    for (int i = 0; i < K_COUNT; ++i) {
        g->timing.ms[i] = 0;
        g->timing.launches[i] = 0;
    }
    if (n_kernels) *n_kernels = K_COUNT;
    return RS_OK;
}

}  // extern "C"
