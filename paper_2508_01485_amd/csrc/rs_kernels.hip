// rs_kernels.hip -- HIP kernels of the robust-spanner scoring pass (gfx950, wave64).
//
// One pass (rs_score):
//   k_rows   Algorithm 1 Steps 1-2 fused, per vertex: run-length count the
//            neighbours' communities into interaction-matrix records
//            (rows are community-sorted, so every community is one run),
//            detect the border vertex, compute every record's weight with
//            Algorithm 2's shared terms (Eq. H_optimal) and the vertex's
//            own-community weight, and a per-block maximum for w_max.
//   k_mid    reduce the per-block maxima to w_max (per graph for a batch; the
//            other totals are reduced when a reader asks), build the big hubs'
//            neighbour filters and, where runs are long, the type-II values.
//   k_score  Eq. RSI per border vertex u, one lane per pair (u, w) with w a
//            foreign neighbour, in the per-(vertex, community) factorised form
//            of Lemmas 1-2 (Section IV, Step 3).  One owner per vertex, fixed
//            summation order, no floating-point atomics.  k_hub_sum adds each
//            hub's chunk partials.
// Top-k (Algorithm 1 Step 4) is an exact radix select on the 96-bit key
// (score bits, complement of the caller id) with 16-bit digits.
//
// Work is cut into static tiles of consecutive vertices (and hub vertices
// with a workgroup each); a launch has one workgroup per tile, so the
// hardware dispatcher balances the uneven tiles.
#include <climits>
#include <cstring>

#include <mutex>

#include "rs_internal.h"

namespace rs {

// ------------------------------------------------------------ helpers
// Blocks for a grid-stride loop over `items`: one per per_block items, at
// least 1 and at most cap.
static inline int grid_for(long long items, int per_block, int cap) {
    long long g = (items + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

__device__ __forceinline__ unsigned long long dbits(double x) { return (unsigned long long)__double_as_longlong(x); }
__device__ __forceinline__ double bitsd(unsigned long long b) { return __longlong_as_double((long long)b); }

// ------------------------------------------------------------ weights
// Eq. H_optimal with Algorithm 2's shared terms: for a vertex of degree d
// whose neighbour-community counts have X = sum f log2 f over ell distinct
// communities, the weight toward a community with count f > 0 is
//   H = -(X - d log2(d - f) - f log2(f / (d - f))) / (d - f),  w = H (ell - 1),
// and toward a community absent from the neighbourhood (f = 0; only the own
// community can be) H = log2 d - X / d with |L| = ell (Eq. weight).
// |L| <= 1 leaves a single community: H = 0 exactly.
__device__ __forceinline__ double flogf(int f);
__device__ __forceinline__ double weight_present(int d, double X, int ell, int f) {
    const int L = ell - 1;
    if (L < 2) return 0.0;
    const double Y = (double)(d - f);
    return (log2(Y) + (flogf(f) - X) / Y) * (double)L;  // = -(X - d log2 Y - f log2(f/Y)) / Y
}

__device__ __forceinline__ double weight_absent(int d, double X, int ell) {
    if (ell < 2) return 0.0;
    const double Y = (double)d;
    return (log2(Y) - X / Y) * (double)ell;
}

__device__ __forceinline__ double flogf(int f) { return f > 1 ? (double)f * log2((double)f) : 0.0; }

// The same terms in a row tile, whose degrees are at most kRowTile: the
// logarithms come from a table in memory (16 KB, made at load with the same
// log2, so the bits are the same), and small arguments (<= kTab; most run
// lengths and degrees) read log2 y, y log2 y and 1/y from LDS.  With the
// logarithms computed in place (and the LDS tables by every workgroup) the row
// pass took 376 against 327 us at n = 3 million, mean degree 30, 87 against 72
// at n = 1 million, mean degree 20, and 73 against 59 at n = 150,000, mean
// degree 71.
constexpr int kTab = 64;
struct Tables {
    double lg[kTab + 1], fl[kTab + 1], rc[kTab + 1];
};
struct TablesMem {
    Tables small;
    double lg[kRowTile + 1];
};
__global__ __launch_bounds__(kBlock) void k_tables(TablesMem *t) {
    for (int i = threadIdx.x; i <= kRowTile; i += kBlock) {
        const double x = (double)i, lg = i > 0 ? log2(x) : 0.0;
        t->lg[i] = lg;
        if (i <= kTab) {
            t->small.lg[i] = lg;
            t->small.fl[i] = flogf(i);
            t->small.rc[i] = i > 0 ? 1.0 / x : 0.0;
        }
    }
}
size_t table_bytes() { return sizeof(TablesMem); }
rs_status launch_tables(rs_graph *g) {
    hipLaunchKernelGGL(k_tables, dim3(1), dim3(kBlock), 0, g->stream, (TablesMem *)g->d.tables);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "table launch");
}

struct Logs {
    const Tables &t;   // LDS
    const double *lg;  // memory: log2 of 1..kRowTile
    __device__ __forceinline__ double flog(int f) const {
        return f <= kTab ? t.fl[f] : (double)f * lg[f];
    }
    __device__ __forceinline__ double present(int d, double X, int ell, int f) const {
        const int L = ell - 1;
        if (L < 2) return 0.0;
        const int Y = d - f;
        if (Y <= kTab) return (t.lg[Y] + (flog(f) - X) * t.rc[Y]) * (double)L;
        return (lg[Y] + (flog(f) - X) / (double)Y) * (double)L;
    }
    __device__ __forceinline__ double absent(int d, double X, int ell) const {
        if (ell < 2) return 0.0;
        if (d <= kTab) return (t.lg[d] - X * t.rc[d]) * (double)ell;
        return (lg[d] - X / (double)d) * (double)ell;
    }
};

// ============================================================ row pass
template <typename OffT>
struct RowArgs {
    const OffT *off;
    const int32_t *deg, *lab;
    const int32_t *clab;  // the community of each entry's neighbour
    const TablesMem *tables;
    const RowTile *tiles;
    const int32_t *hubs;
    int n_tiles, n_hubs, tiles_per_xcd;
    VMeta *meta;
    const int32_t *goff;
    PairRec *prec;     // records at the leader slots, written by this pass
    double *val2;      // scratch of the hub rows here
    const int *blist;  // incremental pass: the listed blocks (k_rows_inc)
    double *wown, *R, *raw;
    double *av;  // [n] a_v = cbrt(own-community weight), dense for the score pass's run sums
    long long *tI, *tII;
    RowPart *part;
    unsigned long long *wmax_part;  // [grid] w_max bits of each block (dense copy for k_mid)
};

struct RowResult {
    int ell, p, q;
    double wown, lmax;
};

struct RowAcc {
    double wmax;
    unsigned long long nb, dp, ell, ellx;
};

// The vertex's row facts of this pass, its own weight and a_v, and zero
// scores for a non-border vertex.
template <typename OffT>
__device__ __forceinline__ void finish_row(const RowArgs<OffT> &A, int v, int d, const RowResult &r, RowAcc &acc) {
    const int fown = r.q - r.p;
    const int dprime = d - fown;
    VMeta m;
    m.deg = d;
    m.ell = r.ell;
    m.p = r.p;
    m.q = r.q;
    A.meta[v] = m;
    A.av[v] = cbrt(r.wown);
    A.wown[v] = r.wown;
    acc.wmax = fmax(acc.wmax, r.lmax);
    acc.ell += (unsigned long long)r.ell;
    acc.ellx += (unsigned long long)(r.ell - (fown > 0 ? 1 : 0));
    if (dprime > 0) {
        acc.nb += 1;
        acc.dp += (unsigned long long)dprime;
    } else {
        A.R[v] = 0.0;
        A.raw[v] = 0.0;
        A.tI[v] = 0;
        A.tII[v] = 0;
    }
}

// Sum over a wavefront's lanes, and maximum of non-negative doubles, in lane 63
// (row shifts and broadcasts: no LDS).
template <int kCtrl, int kRows>
__device__ __forceinline__ int dpp_or_zero(int x) {
    return __builtin_amdgcn_update_dpp(0, x, kCtrl, kRows, 0xf, false);
}
template <int kCtrl, int kRows>
__device__ __forceinline__ double dpp_max(double x) {
    const unsigned long long b = dbits(x);
    const unsigned int lo = (unsigned int)dpp_or_zero<kCtrl, kRows>((int)(unsigned int)b);
    const unsigned int hi = (unsigned int)dpp_or_zero<kCtrl, kRows>((int)(unsigned int)(b >> 32));
    return fmax(x, bitsd(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ unsigned int wave_sum_last(unsigned int v) {
    int x = (int)v;
    x += dpp_or_zero<0x111, 0xf>(x);  // row_shr:1, 2, 4, 8
    x += dpp_or_zero<0x112, 0xf>(x);
    x += dpp_or_zero<0x114, 0xf>(x);
    x += dpp_or_zero<0x118, 0xf>(x);
    x += dpp_or_zero<0x142, 0xa>(x);  // row_bcast:15, 31
    x += dpp_or_zero<0x143, 0xc>(x);
    return (unsigned int)x;
}
__device__ __forceinline__ double wave_max_last(double x) {
    x = dpp_max<0x111, 0xf>(x);
    x = dpp_max<0x112, 0xf>(x);
    x = dpp_max<0x114, 0xf>(x);
    x = dpp_max<0x118, 0xf>(x);
    x = dpp_max<0x142, 0xa>(x);
    return dpp_max<0x143, 0xc>(x);
}

// A row block's totals: a hub's are its first thread's already; a tile's
// counts fit 16 bits each (kRowTile entries), so they are summed two to a
// register (five 64-bit shuffled reductions took an eighth of the pass).
__device__ __forceinline__ void store_row_part(const RowPart &p, RowPart *out, unsigned long long *wmax_out) {
    *out = p;
    *wmax_out = p.wmax_bits;
}
__device__ __forceinline__ void hub_row_part(const RowAcc &acc, RowPart *out, unsigned long long *wmax_out) {
    if (threadIdx.x != 0) return;
    RowPart p = {};
    p.wmax_bits = dbits(acc.wmax);
    p.n_border = acc.nb;
    p.sum_dprime = acc.dp;
    p.sum_ell = acc.ell;
    p.sum_ell_x = acc.ellx;
    store_row_part(p, out, wmax_out);
}
static_assert(kRowTile < 65536 && kRowTileV < 65536, "a tile's counts fit 16 bits");
__device__ __forceinline__ void block_reduce_row(const RowAcc &acc, RowPart *out, unsigned long long *wmax_out) {
    __shared__ double s_w[kBlock / 64];
    __shared__ unsigned int s_u[2][kBlock / 64];
    const double w = wave_max_last(acc.wmax);
    const unsigned int a = wave_sum_last((unsigned int)acc.nb | (unsigned int)acc.dp << 16);
    const unsigned int b = wave_sum_last((unsigned int)acc.ell | (unsigned int)acc.ellx << 16);
    if ((threadIdx.x & 63) == 63) {
        s_w[threadIdx.x >> 6] = w;
        s_u[0][threadIdx.x >> 6] = a;
        s_u[1][threadIdx.x >> 6] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        RowPart p = {};
        for (int i = 0; i < kBlock / 64; ++i) {
            p.wmax_bits = max(p.wmax_bits, dbits(s_w[i]));
            p.n_border += s_u[0][i] & 0xffffu;
            p.sum_dprime += s_u[0][i] >> 16;
            p.sum_ell += s_u[1][i] & 0xffffu;
            p.sum_ell_x += s_u[1][i] >> 16;
        }
        store_row_part(p, out, wmax_out);
    }
}

// Tile of the grid's block b: hubs take the first blocks; the tiles follow,
// the tiles of one XCD contiguous (blocks are dealt to the XCDs round-robin,
// so block b runs on XCD b % 8 and consecutive tiles share that XCD's L2).
__device__ __forceinline__ int tile_of_block(int b, int n_hubs, int per_xcd) {
    return (b & 7) * per_xcd + ((b - n_hubs) >> 3);
}

// ------------------------------------------------------------ row tiles
// A row tile is a run of consecutive vertices whose rows (capacity <=
// kRowTile entries, a contiguous slice of col) are processed flat:
//   1. every entry's neighbour community is read from clab (coalesced);
//   2. an entry starts a run if it starts a row or its label differs from
//      the previous entry's (rows are community-sorted, so each run is one
//      interaction-matrix record); run starts are ranked with wavefront
//      ballots and a block prefix;
//   3. flat over the runs: the own community's run, or where it would be, and
//      which runs are longer than one (a bit each);
//   4. one thread per vertex adds X = sum f log2 f over those in run order (a
//      run of one adds zero) and has ell, p, q from the run indices;
//   5. the records' weights (Eq. H_optimal) are computed flat over runs.
// One lane walking all of its vertex's runs held its wavefront for a third of
// the kernel: a tile has some 75 to 110 vertices and ten times the runs.  With
// the block totals below: n = 3 million, mean degree 30, 467 -> 376 us; n = 1
// million, mean degree 20, 104 -> 87; n = 150,000, mean degree 71, 92 -> 73;
// 128 graphs 150 -> 123.
// A removed entry is -1 (after compaction): such a tail forms a run that is
// skipped.
constexpr int kRowW = kBlock / 64;      // wavefronts per workgroup
constexpr int kRowU = kRowTile / kBlock; // entries per thread
constexpr int kRowM = kRowTile / 64;     // ballot words per tile
static_assert(kRowTile % kBlock == 0 && kRowTile <= 65535 && kRowTileV % kBlock == 0, "row tile size");

// Streaming state of a hub row (one workgroup).
struct HubSeg {
    int prev, next_prev;                     // label before the segment / of its last entry
    int open_start, open_label;              // run open at the segment boundary (open_start < 0: none)
    int nruns;                               // runs started before the segment
    int own;                                 // 1 once the own community's run has started
    double red[kRowW];
    int ired[kRowW];
};

struct RowTileShared {
    HubSeg hub;
    Tables tab;
    unsigned long long bm[kRowM];        // row-start bits
    unsigned long long mask[kRowM];      // run-start bits; then, by run, those longer than one
    int mbase[kRowM];                    // run starts before each mask word
    unsigned short rbase[kRowM];         // row starts before each 64 entries
    int wlast[kRowW], wcnt[kRowW], wrow[kRowW];
    unsigned short runpos[kRowTile + 1]; // tile-local entry of each run start (+ end)
    unsigned short runv[kRowTile];       // row of each run (the tile's rows with a capacity, in order)
    int runlab[kRowTile];                // label of each run (-1: removed tail)
    union {  // by row
        int vlab[2 * kRowTileV];  // its community, until X is known
        double vX[kRowTileV];
    };
    unsigned int vde[kRowTileV];     // degree and ell (16 bits each)
    short vslot[kRowTileV];          // tile slot of a foreign entry below the own community, minus its tile-local entry
    unsigned short vrun[kRowTileV];  // first run not below the own community, and kOwnRun when that is the own one
};
constexpr int kOwnRun = 0x8000;
// A workgroup takes 26.9 KB, so six share a CU (with the facts unpacked, five).
static_assert(6 * sizeof(RowTileShared) <= 160 * 1024, "six row workgroups per CU");

__device__ __forceinline__ int run_index(const RowTileShared &S, int e) {
    return S.mbase[e >> 6] + __popcll(S.mask[e >> 6] & ((1ull << (e & 63)) - 1ull));
}

// X of one row with the whole wavefront, for rows with many runs longer than
// one, where one lane's sum keeps the other 63 waiting: the terms 64 runs at a
// time, added in run order, as the single lane does.
// (6, 12 or 24 as the limit: the same within 2 %.)
constexpr int kWalkRuns = 12;
__device__ __forceinline__ double lane_value(double x, int l) {
    const unsigned long long b = dbits(x);
    const unsigned int lo = __builtin_amdgcn_readlane((int)(unsigned int)b, l);
    const unsigned int hi = __builtin_amdgcn_readlane((int)(unsigned int)(b >> 32), l);
    return bitsd(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double wave_walk(const RowTileShared &S, const Logs &logs, int rf, int re, int lane) {
    double x = 0.0;
    for (int r0 = rf; r0 < re; r0 += 64) {
        const int r = r0 + lane;
        int f = 0;
        if (r < re && ((S.mask[r >> 6] >> (r & 63)) & 1ull)) f = (int)S.runpos[r + 1] - (int)S.runpos[r];
        const double t = f > 1 ? logs.flog(f) : 0.0;
        for (unsigned long long m = __ballot(f > 1); m; m &= m - 1ull) x += lane_value(t, __ffsll((long long)m) - 1);
    }
    return x;
}

template <typename OffT>
__device__ void row_tile(const RowArgs<OffT> &A, RowTileShared &S, int t, RowAcc &acc) {
    constexpr int kVU = kRowTileV / kBlock;  // vertices per thread
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const RowTile tl = A.tiles[t];
    const int v0 = tl.v0, nv = tl.v1 - tl.v0;
    const OffT e0 = (OffT)tl.e0;
    const int TE = tl.te;
    const int go0 = A.goff[v0];
    if (tid < kRowM) S.bm[tid] = 0ull;
    // the tile's entries and the facts of this thread's vertices, all
    // independent loads issued together
    int L[kRowU];
#pragma unroll
    for (int i = 0; i < kRowU; ++i) {
        const int e = wave * (kRowTile / kRowW) + i * 64 + lane;
        L[i] = e < TE ? A.clab[e0 + e] : -2;
    }
    int vo[kVU], vc[kVU], vdeg[kVU], vlab[kVU];
    int vgo[kVU];
#pragma unroll
    for (int j = 0; j < kVU; ++j) {
        // a slot past the tile loads the tile's first vertex (tiles are never
        // empty), and every use below skips it: no branch around the loads,
        // which would wait for them before the next slot's
        const int i = tid + j * kBlock;
        const int ic = i < nv ? i : 0;
        const OffT a0 = A.off[v0 + ic], a1 = A.off[v0 + ic + 1];
        vo[j] = (int)(a0 - e0);
        vc[j] = (int)(a1 - a0);
        vdeg[j] = A.deg[v0 + ic];
        vlab[j] = A.lab[v0 + ic];
        vgo[j] = A.goff[v0 + ic];
    }
    constexpr int kTabN = (int)(sizeof(Tables) / sizeof(double));
    static_assert(kTabN <= kBlock, "a table entry per thread");
    const double te = ((const double *)&A.tables->small)[min(tid, kTabN - 1)];
    if (tid < kTabN) ((double *)&S.tab)[tid] = te;
    const Logs logs = {S.tab, A.tables->lg};
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kVU; ++j)
        if (tid + j * kBlock < nv && vc[j] > 0) atomicOr(&S.bm[vo[j] >> 6], 1ull << (vo[j] & 63));
    if (lane == 63) S.wlast[wave] = L[kRowU - 1];
    __syncthreads();
    unsigned long long m[kRowU], rows[kRowU];
    int cnt = 0, nrow = 0;
#pragma unroll
    for (int i = 0; i < kRowU; ++i) {
        const int e = wave * (kRowTile / kRowW) + i * 64 + lane;
        int lp = __shfl_up(L[i], 1);
        const int carry = i > 0 ? __shfl(L[i > 0 ? i - 1 : 0], 63) : (wave > 0 ? S.wlast[wave > 0 ? wave - 1 : 0] : INT_MIN);
        if (lane == 0) lp = carry;
        rows[i] = S.bm[e >> 6];
        m[i] = __ballot(e < TE && (((rows[i] >> lane) & 1ull) || L[i] != lp));
        cnt += __popcll(m[i]);
        nrow += __popcll(rows[i]);
    }
    if (lane == 0) {
        S.wcnt[wave] = cnt;
        S.wrow[wave] = nrow;
    }
    __syncthreads();
    int base = 0, total = 0, row0 = 0;
#pragma unroll
    for (int x = 0; x < kRowW; ++x) {
        const int c = S.wcnt[x];
        if (x < wave) {
            base += c;
            row0 += S.wrow[x];
        }
        total += c;
    }
    const unsigned long long lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int i = 0; i < kRowU; ++i) {
        const int e = wave * (kRowTile / kRowW) + i * 64 + lane;
        if (lane == 0) {
            S.mask[e >> 6] = m[i];
            S.mbase[e >> 6] = base;
            S.rbase[e >> 6] = (unsigned short)row0;
        }
        if ((m[i] >> lane) & 1ull) {
            const int r = base + __popcll(m[i] & lt);
            S.runpos[r] = (unsigned short)e;
            S.runlab[r] = L[i];
            // (the tile's first entry starts a row, so the count is not 0)
            S.runv[r] = (unsigned short)(row0 + __popcll(rows[i] & (lt << 1 | 1ull)) - 1);
        }
        base += __popcll(m[i]);
        row0 += __popcll(rows[i]);
    }
    if (tid == 0) S.runpos[total] = (unsigned short)TE;
    __syncthreads();
    // each vertex's runs [rf, re) and its row; until a run says more, the own
    // community's place is before them
    int vrf[kVU], vre[kVU], vk[kVU];
#pragma unroll
    for (int j = 0; j < kVU; ++j) {
        vrf[j] = vre[j] = vk[j] = 0;
        if (tid + j * kBlock < nv && vc[j] > 0) {
            const int o = vo[j], c = vc[j];
            vrf[j] = run_index(S, o);
            vre[j] = o + c >= TE ? total : run_index(S, o + c);
            vk[j] = (int)S.rbase[o >> 6] + __popcll(S.bm[o >> 6] & ((1ull << (o & 63)) - 1ull));
            S.vrun[vk[j]] = (unsigned short)vrf[j];
            S.vlab[vk[j]] = vlab[j];
        }
    }
    __syncthreads();
    for (int r0 = wave * 64; r0 < total; r0 += kBlock) {
        const int r = r0 + lane;
        bool more = false;
        if (r < total) {
            const int lb = S.runlab[r], q = S.runv[r];
            more = lb >= 0 && (int)S.runpos[r + 1] - (int)S.runpos[r] > 1;
            const int cv = S.vlab[q];
            if (lb == cv) {
                S.vrun[q] = (unsigned short)(r | kOwnRun);
            } else if (lb >= 0 && lb < cv) {  // the last run below the own community, if that has none
                const int ln = r + 1 < total && S.runv[r + 1] == q ? S.runlab[r + 1] : -1;
                if (ln < 0 || ln > cv) S.vrun[q] = (unsigned short)(r + 1);
            }
        }
        const unsigned long long f1 = __ballot(more);
        if (lane == 0) S.mask[r0 >> 6] = f1;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kVU; ++j) {
        if (__ballot(tid + j * kBlock < nv) == 0ull) break;  // no vertex in this wavefront
        const int i = tid + j * kBlock;
        const bool in = i < nv;
        const int o = vo[j], c = in ? vc[j] : 0, d = vdeg[j], k = vk[j];
        const int rf = vrf[j], re = vre[j];
        double X = 0.0;
        int ell = 0, vr = 0;
        bool own = false, far = false;
        if (c > 0) {
            ell = re - rf - (S.runlab[re - 1] < 0 ? 1 : 0);  // (a removed tail is the last run)
            vr = S.vrun[k] & (kOwnRun - 1);
            own = (S.vrun[k] & kOwnRun) != 0;
            // at most 64 runs lie in two words
            far = re - rf > 64;
            if (!far) {
                unsigned long long w0 = S.mask[rf >> 6] >> (rf & 63);
                if ((rf & 63) != 0 && (rf >> 6) < (re - 1) >> 6) w0 |= S.mask[(rf >> 6) + 1] << (64 - (rf & 63));
                if (re - rf < 64) w0 &= (1ull << (re - rf)) - 1ull;
                far = __popcll(w0) > kWalkRuns;
                if (!far)
                    for (; w0; w0 &= w0 - 1ull) {
                        const int r = rf + __ffsll((long long)w0) - 1;
                        X += logs.flog((int)S.runpos[r + 1] - (int)S.runpos[r]);
                    }
            }
        }
        for (unsigned long long pend = __ballot(far); pend; pend &= pend - 1ull) {
            const int l = __ffsll((long long)pend) - 1;
            const double x = wave_walk(S, logs, __builtin_amdgcn_readlane(rf, l), __builtin_amdgcn_readlane(re, l), lane);
            if (lane == l) X = x;
        }
        if (!in) continue;
        // the runs below the own community come first
        const int below = c > 0 ? (int)S.runpos[vr] - o : 0;
        const int fown = own ? (int)S.runpos[vr + 1] - (int)S.runpos[vr] : 0;
        if (c > 0) {
            S.vX[k] = X;
            S.vde[k] = (unsigned int)d | (unsigned int)ell << 16;
            S.vslot[k] = (short)(vgo[j] - go0 - o);
        }
        RowResult res;
        res.ell = ell;
        res.p = below;
        res.q = below + fown;
        res.wown = fown > 0 ? logs.present(d, X, ell, fown) : logs.absent(d, X, ell);
        res.lmax = res.wown;
        finish_row(A, v0 + i, d, res, acc);
    }
    __syncthreads();
    // a foreign run's record goes to its leader slot; the own community's
    // weight is the vertex's own weight already
    for (int r = tid; r < total; r += kBlock) {
        const int lb = S.runlab[r];
        if (lb < 0) continue;
        const int i = S.runv[r];
        const int vr = S.vrun[i] & (kOwnRun - 1);
        const bool own = (S.vrun[i] & kOwnRun) != 0;
        if (own && r == vr) continue;
        const int p0 = (int)S.runpos[r];
        const unsigned int de = S.vde[i];
        PairRec pr;
        pr.f = (int)S.runpos[r + 1] - p0;
        pr.w = logs.present((int)(de & 0xffffu), S.vX[i], (int)(de >> 16), pr.f);
        pr.c = lb;
        const int fo = own && r > vr ? (int)S.runpos[vr + 1] - (int)S.runpos[vr] : 0;
        const int s = go0 + S.vslot[i] + p0 - fo;
        const int f = pr.f;
        A.prec[s] = pr;
        for (int t = 1; t < f; ++t) {
            pr.f = -t;
            A.prec[s + t] = pr;
        }
        acc.wmax = fmax(acc.wmax, pr.w);
    }
}

// ------------------------------------------------------------ hub rows
// A vertex whose row capacity exceeds kRowTile gets a workgroup.  Its row is
// streamed once in segments of kRowTile entries with the tile's flat machinery
// (labels, run starts by ballot, runs closed flat over LDS; the next segment's
// labels are in flight meanwhile): this counts the runs, X and the own run and
// lists the foreign runs' starts.  The run still open at a segment's end is
// carried to the next.  The records are then computed flat over the list.
// Streaming the row a second time for the records, with one thread writing
// all slots of a run, took a hub of 46,000 neighbours 660 us, longer than all
// row tiles of n = 3 million.
struct HubRun {
    int start;  // row position
    int label;
};
template <typename OffT>
__device__ void hub_stream(const RowArgs<OffT> &A, RowTileShared &S, OffT rb, int d, int cv, HubRun *list,
                           double &xpart, int &below, int &fown) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    HubSeg &H = S.hub;
    if (tid == 0) {
        H.prev = INT_MIN;
        H.open_start = -1;
        H.nruns = 0;
        H.own = 0;
    }
    auto close = [&](int label, int f) {
        xpart += flogf(f);
        if (label == cv)
            fown = f;
        else if (label < cv)
            below += f;
    };
    const int e0 = wave * (kRowTile / kRowW) + lane;
    int L[kRowU];
#pragma unroll
    for (int i = 0; i < kRowU; ++i) L[i] = A.clab[rb + min(e0 + i * 64, max(d - 1, 0))];
    for (int seg0 = 0; seg0 < d; seg0 += kRowTile) {
        const int TE = min(kRowTile, d - seg0);
        int next[kRowU];
#pragma unroll
        for (int i = 0; i < kRowU; ++i) next[i] = A.clab[rb + min(seg0 + kRowTile + e0 + i * 64, d - 1)];
        __syncthreads();  // the previous segment is done with S
        if (lane == 63) S.wlast[wave] = L[kRowU - 1];
#pragma unroll
        for (int i = 0; i < kRowU; ++i)
            if (e0 + i * 64 == TE - 1) H.next_prev = L[i];
        __syncthreads();
        unsigned long long m[kRowU];
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < kRowU; ++i) {
            int lp = __shfl_up(L[i], 1);
            const int carry = i > 0 ? __shfl(L[i > 0 ? i - 1 : 0], 63) : (wave > 0 ? S.wlast[wave > 0 ? wave - 1 : 0] : H.prev);
            if (lane == 0) lp = carry;
            m[i] = __ballot(e0 + i * 64 < TE && L[i] != lp);
            cnt += __popcll(m[i]);
        }
        if (lane == 0) S.wcnt[wave] = cnt;
        __syncthreads();
        int base = 0, total = 0;
#pragma unroll
        for (int x = 0; x < kRowW; ++x) {
            const int c = S.wcnt[x];
            if (x < wave) base += c;
            total += c;
        }
        const unsigned long long lt = (1ull << lane) - 1ull;
#pragma unroll
        for (int i = 0; i < kRowU; ++i) {
            if ((m[i] >> lane) & 1ull) {
                const int r = base + __popcll(m[i] & lt);
                S.runpos[r] = (unsigned short)(e0 + i * 64);
                S.runlab[r] = L[i];
                if (L[i] == cv) H.own = 1;
            }
            base += __popcll(m[i]);
        }
        if (tid == 0) S.runpos[total] = (unsigned short)TE;
        __syncthreads();
        const bool last = seg0 + TE >= d;
        const int nr0 = H.nruns;
        // the run carried from the previous segment closes at this segment's
        // first run start (or at the row's end)
        if (tid == 0 && H.open_start >= 0 && (total > 0 || last)) {
            const int end = total > 0 ? seg0 + (int)S.runpos[0] : d;
            close(H.open_label, end - H.open_start);
            H.open_start = -1;
        }
        const int closed = last ? total : total - 1;  // the segment's last run stays open unless the row ends
        for (int r = tid; r < total; r += kBlock) {
            const int lb = S.runlab[r], p0 = (int)S.runpos[r];
            if (r < closed) close(lb, (int)S.runpos[r + 1] - p0);
            if (lb != cv) list[nr0 + r - (lb > cv ? H.own : 0)] = HubRun{seg0 + p0, lb};
        }
        __syncthreads();
        if (tid == 0) {
            if (!last && total > 0) {
                H.open_start = seg0 + (int)S.runpos[total - 1];
                H.open_label = S.runlab[total - 1];
            }
            H.nruns = nr0 + total;
            H.prev = H.next_prev;
        }
#pragma unroll
        for (int i = 0; i < kRowU; ++i) L[i] = next[i];
    }
    __syncthreads();
}

__device__ __forceinline__ double block_sum_d(double x, double *red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < kRowW; ++i) t += red[i];
    __syncthreads();
    return t;
}

__device__ __forceinline__ double block_max_d(double x, double *red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < kRowW; ++i) t = fmax(t, red[i]);
    __syncthreads();
    return t;
}

__device__ __forceinline__ int block_sum_i(int x, int *red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    int t = 0;
    for (int i = 0; i < kRowW; ++i) t += red[i];
    __syncthreads();
    return t;
}

template <typename OffT>
__device__ void hub_row(const RowArgs<OffT> &A, RowTileShared &S, int v, RowAcc &acc) {
    const OffT rb = A.off[v];
    const int d = A.deg[v];
    const int cv = A.lab[v];
    double xpart = 0.0, lmax = 0.0;
    int below = 0, fown = 0;
    const int go = A.goff[v];
    HubRun *list = (HubRun *)(A.val2 + go);  // the type-II values are written after this pass
    hub_stream(A, S, rb, d, cv, list, xpart, below, fown);
    const double X = block_sum_d(xpart, S.hub.red);
    const int p = block_sum_i(below, S.hub.ired);
    const int fo = block_sum_i(fown, S.hub.ired);  // one thread holds the own run's length
    const int ell = S.hub.nruns;
    const int nf = ell - (fo > 0 ? 1 : 0);
    const int lane = threadIdx.x & 63;
    for (int r0 = (int)threadIdx.x - lane; r0 < nf; r0 += kBlock) {
        const int r = r0 + lane;
        PairRec pr = {0.0, 0, 0};
        int s = 0;
        if (r < nf) {
            const HubRun h = list[r];
            int end = r + 1 < nf ? list[r + 1].start : d;
            if (h.start < p) end = min(end, p);  // the own run lies between
            pr.f = end - h.start;
            pr.c = h.label;
            pr.w = weight_present(d, X, ell, pr.f);
            s = go + h.start - (h.label > cv ? fo : 0);
            A.prec[s] = pr;
            lmax = fmax(lmax, pr.w);
        }
        // the other slots of the lanes' runs, one run at a time
        for (unsigned long long m = __ballot(pr.f > 1); m; m &= m - 1ull) {
            const int l = __ffsll((long long)m) - 1;
            const int f = __builtin_amdgcn_readlane(pr.f, l), s0 = __builtin_amdgcn_readlane(s, l);
            PairRec q;
            q.w = lane_value(pr.w, l);
            q.c = __builtin_amdgcn_readlane(pr.c, l);
            for (int t = 1 + lane; t < f; t += 64) {
                q.f = -t;
                A.prec[s0 + t] = q;
            }
        }
    }
    const double lm = block_max_d(lmax, S.hub.red);
    if (threadIdx.x == 0) {
        RowResult r;
        r.ell = ell;
        r.p = p;
        r.q = p + fo;
        r.wown = fo > 0 ? weight_present(d, X, ell, fo) : weight_absent(d, X, ell);
        r.lmax = fmax(lm, r.wown);
        finish_row(A, v, d, r, acc);
    }
}

// Reduce the row partials of a pass into the counters (one workgroup; the
// loads of four partials per thread are in flight together).
__device__ void reduce_row_parts(const RowPart *part, int np, DevCounters *c) {
    __shared__ unsigned long long s[5][kBlock / 64];
    unsigned long long w = 0, nb = 0, dp = 0, ell = 0, ellx = 0;
    for (int i0 = threadIdx.x; i0 < np; i0 += 4 * kBlock) {
        RowPart q[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = i0 + j * kBlock;
            if (i < np) {
                q[j] = part[i];
            } else {
                q[j] = RowPart{};
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            w = max(w, q[j].wmax_bits);
            nb += q[j].n_border;
            dp += q[j].sum_dprime;
            ell += q[j].sum_ell;
            ellx += q[j].sum_ell_x;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        w = max(w, (unsigned long long)__shfl_xor(w, o));
        nb += __shfl_xor(nb, o);
        dp += __shfl_xor(dp, o);
        ell += __shfl_xor(ell, o);
        ellx += __shfl_xor(ellx, o);
    }
    if ((threadIdx.x & 63) == 0) {
        s[0][threadIdx.x >> 6] = w;
        s[1][threadIdx.x >> 6] = nb;
        s[2][threadIdx.x >> 6] = dp;
        s[3][threadIdx.x >> 6] = ell;
        s[4][threadIdx.x >> 6] = ellx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        DevCounters r = *c;
        r.wmax_bits = r.n_border = r.sum_dprime = r.sum_ell = r.sum_ell_x = 0;
        for (int i = 0; i < kBlock / 64; ++i) {
            r.wmax_bits = max(r.wmax_bits, s[0][i]);
            r.n_border += s[1][i];
            r.sum_dprime += s[2][i];
            r.sum_ell += s[3][i];
            r.sum_ell_x += s[4][i];
        }
        *c = r;
    }
}

// Algorithm 1 Steps 1-2 for every vertex: hub rows first, then the tiles.
template <typename OffT>
__global__ __launch_bounds__(kBlock, 6) void k_rows(RowArgs<OffT> A) {
    __shared__ RowTileShared S;
    RowAcc acc = {0.0, 0, 0, 0, 0};
    const int b = (int)blockIdx.x;
    if (b < A.n_hubs) {
        hub_row(A, S, A.hubs[b], acc);
        hub_row_part(acc, &A.part[b], &A.wmax_part[b]);
    } else {
        const int t = tile_of_block(b, A.n_hubs, A.tiles_per_xcd);
        if (t < A.n_tiles) row_tile(A, S, t, acc);
        block_reduce_row(acc, &A.part[b], &A.wmax_part[b]);
    }
}

// Whether an incremental pass runs every block of the full launches: its
// units (listed row blocks, main score blocks and big-hub chunks, and the
// units of the affected tile vertices) exceed kFullPassTenths of the full
// pass's workgroups (a removed hub touches much of the graph; full launches
// run faster per unit, and the bits are the same).  Every kernel of the
// pass decides alike from the marks' counters.
__device__ __forceinline__ bool inc_full(const unsigned long long *ictr, int grid_rows, int grid_score) {
    long long u = (long long)ictr[kIcRows] + (long long)ictr[kIcMain] + (long long)ictr[kIcBig];
#pragma unroll
    for (int b = 0; b < kScoreBins; ++b) u += ((long long)ictr[kIcBins + b] + (kBlock >> b) - 1) / (kBlock >> b);
    return 10 * u > (long long)kFullPassTenths * ((long long)grid_rows + grid_score);
}

// The incremental pass's row blocks: block i of a capped grid takes the
// listed blocks i, i + gridDim.x, ... (every block of the full launch in a
// full pass), each exactly as k_rows runs it.
template <typename OffT>
__global__ __launch_bounds__(kBlock) void k_rows_inc(RowArgs<OffT> A, const unsigned long long *ictr, int grid_rows,
                                                     int grid_score) {
    __shared__ RowTileShared S;
    const bool full = inc_full(ictr, grid_rows, grid_score);
    const long long cnt = full ? (long long)grid_rows : (long long)ictr[kIcRows];
    for (long long i = blockIdx.x; i < cnt; i += gridDim.x) {
        RowAcc acc = {0.0, 0, 0, 0, 0};
        const int b = full ? (int)i : A.blist[i];
        if (b < A.n_hubs) {
            hub_row(A, S, A.hubs[b], acc);
            hub_row_part(acc, &A.part[b], &A.wmax_part[b]);
        } else {
            const int t = tile_of_block(b, A.n_hubs, A.tiles_per_xcd);
            if (t < A.n_tiles) row_tile(A, S, t, acc);
            block_reduce_row(acc, &A.part[b], &A.wmax_part[b]);
        }
        __syncthreads();  // the next block's LDS
    }
}

// w_max of a pass from the dense per-block maxima of the row kernel (part of
// k_mid): up to kWmaxBlocks workgroups of 1,024 threads each take a contiguous slice
// (eight loads per thread in flight together) and store its maximum; the
// workgroup that finishes last (a ticket) takes the maximum of those and
// resets the ticket.  A maximum does not depend on the order, so the bits are
// those of a single workgroup's.  The other row totals are reduced only when
// a reader asks for them.
constexpr int kWmaxBlocks = 64;
constexpr int kMidThreads = 1024;
__device__ __forceinline__ void reduce_wmax(const unsigned long long *wpart, int np, int block, int blocks,
                                            unsigned long long *wblk, unsigned int *ticket, DevCounters *c) {
    __shared__ unsigned long long s[kMidThreads / 64];
    const int per = (np + blocks - 1) / blocks;
    const int lo = block * per, hi = min(np, lo + per);
    unsigned long long w = 0;
    for (int i0 = lo + threadIdx.x; i0 < hi; i0 += 8 * kMidThreads) {
        unsigned long long q[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int i = i0 + j * kMidThreads;
            q[j] = i < hi ? wpart[i] : 0ull;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) w = max(w, q[j]);
    }
    for (int o = 32; o > 0; o >>= 1) w = max(w, (unsigned long long)__shfl_xor(w, o));
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = w;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long m = 0;
        for (int i = 0; i < kMidThreads / 64; ++i) m = max(m, s[i]);
        bool last = true;
        if (blocks > 1) {
            wblk[block] = m;
            __threadfence();
            last = atomicAdd(ticket, 1u) == (unsigned int)blocks - 1u;
            if (last) {
                __threadfence();
                for (int i = 0; i < blocks; ++i) m = max(m, ((volatile unsigned long long *)wblk)[i]);
                *ticket = 0u;
            }
        }
        if (last) c->wmax_bits = m;
    }
}

// Batched graphs: each graph's w_max, the maximum of the w_max of its row
// blocks (row tiles never span two graphs), one wavefront per graph.  The
// block values are fp64 bits maximised as integers, as for the whole-graph
// w_max, so a graph's w_max has the bits it has when the graph is alone.
__device__ __forceinline__ void reduce_wmax_graph(const unsigned long long *wpart, const int32_t *gblk_off,
                                                  const int32_t *gblk, int gi, unsigned long long *gwmax) {
    const int lane = threadIdx.x & 63;
    unsigned long long m = 0;
    for (int i = gblk_off[gi] + lane; i < gblk_off[gi + 1]; i += 64) m = max(m, wpart[gblk[i]]);
    for (int o = 32; o > 0; o >>= 1) m = max(m, (unsigned long long)__shfl_xor(m, o));
    if (lane == 0) gwmax[gi] = m;
}

// All row totals of the last pass (for the counter readers).
__global__ __launch_bounds__(kBlock) void k_reduce_rows(const RowPart *part, int np, DevCounters *c) {
    reduce_row_parts(part, np, c);
}

// ============================================================ score pass
struct ScoreArgs {
    const int32_t *goff, *fcol;  // slots of the foreign entries and their neighbours
    const uint8_t *sown;         // a tile slot's vertex (index in the tile)
    const int2 *tiles;
    const int32_t *hubs;
    int n_tiles, n_hubs, tiles_per_xcd;
    const int32_t *hub_first;
    const int2 *hub_chunk;
    int n_chunks, n_chunks_lds;
    HubPart *hub_part;
    const int32_t *outl;
    const int64_t *oo;      // out-list offsets
    const VMeta *meta;
    const PairRec *prec;    // records at the leader slots, written by the row pass
    const uint32_t *hfilter;  // big hubs' neighbour filters (hub n_hubs_lds + i at i * kFilterWords)
    const OutEnt *oe;         // each out-list entry's leader slots
    int n_hubs_lds;
    const PairLink *plink;  // the links of the slots
    const double *av;       // [n] a_v of the row pass
    const double *val2;     // the slots' type-II values (k_mid), or null: each pair sums its run
    const unsigned long long *gwmax;  // batched graphs: w_max bits of each graph, else null
    const int32_t *vgraph;            // batched graphs: graph of each vertex
    double *R, *raw;
    long long *tI, *tII;
    const DevCounters *ctr;
};

// The first position in the sorted a[lo, hi) in LDS that holds x or more.
__device__ __forceinline__ int lds_lower(const int *a, int lo, int hi, int x) {
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < x)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Out-lists keep removed entries complemented (~id) in place, so a list is
// ascending in the decoded id.
__device__ __forceinline__ int out_id(int x) { return x < 0 ? ~x : x; }

// Position of the live id x among the n out-list entries a[0..n) in LDS, or -1.
__device__ __forceinline__ int lds_find_out(const int *a, int n, int x) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (out_id(a[mid]) < x)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo < n && a[lo] == x ? lo : -1;
}

// Position of the live id t in the sorted out-list outl[o0, o1) in HBM
// (removed ids are complemented and keep their place), or -1: a 16-ary
// search on the decoded ids, each step 15 loads issued together (a list of up
// to 16 entries is one step).  Probes past the range load its last entry and
// are discarded after the load: a test before the load would make each
// probe wait for the previous one.
__device__ __forceinline__ long long out_find(const int32_t *outl, long long o0, long long o1, int t) {
    long long lo = o0, hi = o1;
    if (hi <= lo) return -1;
    while (hi - lo > 16) {
        const long long st = (hi - lo + 15) >> 4;
        int y[15];
#pragma unroll
        for (int j = 1; j < 16; ++j) y[j - 1] = outl[min(lo + j * st, hi - 1)];
        int cnt = 0;
#pragma unroll
        for (int j = 1; j < 16; ++j) cnt += (int)((lo + j * st < hi) & (out_id(y[j - 1]) <= t));
        lo += cnt * st;
        hi = min(hi, lo + st);
    }
    int y[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) y[j] = outl[min(lo + j, hi - 1)];
    long long f = -1;
#pragma unroll
    for (int j = 0; j < 16; ++j)
        if (lo + j < hi && y[j] == t) f = lo + j;
    return f;
}

// The type-II terms of the pair (u, w), w a foreign neighbour of u (Lemma 2,
// unnormalised weights), from w's record for C(u) (W = w_w(C(u)) and the run
// of C(u) in w's list from its leader slot on): W^(2/3) times the sum of a_v
// over the other members v of that run (v in C(u), v adjacent to w; counted
// whether or not v ~ u), and the count f_w(C(u)) - 1.
// val2 holds the same sums, in the same order, when k_mid computed them.
__device__ __forceinline__ double type2_pair(const ScoreArgs &A, int u, const PairRec &pr, const PairLink &pl) {
    if (pr.f <= 1) return 0.0;
    if (A.val2) return A.val2[pl.slot];
    const int lead = pl.lead;
    double S = 0.0;
    const int32_t *run = A.fcol + lead;
    for (int i = 0; i < pr.f; i += 8) {
        int x[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) x[t] = i + t < pr.f ? run[i + t] : u;
        double av[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) av[t] = x[t] != u ? A.av[x[t]] : 0.0;
#pragma unroll
        for (int t = 0; t < 8; ++t) S += av[t];
    }
    const double c1 = cbrt(pr.w);
    return c1 * c1 * S;
}

// R of Algorithm 1: the raw sum over w_max and d(d-1); 0 when d < 2 or w_max = 0.
__device__ __forceinline__ double score_value(double acc, int d, double wmax) {
    return (d >= 2 && wmax > 0.0) ? acc / wmax / (double)((long long)d * (d - 1)) : 0.0;
}

__device__ __forceinline__ void score_store(const ScoreArgs &A, int u, int d, double acc, long long cI,
                                            long long cII, double wmax) {
    A.R[u] = score_value(acc, d, A.gwmax ? bitsd(A.gwmax[A.vgraph[u]]) : wmax);
    A.raw[u] = acc;
    A.tI[u] = cI;
    A.tII[u] = cII;
}

// Exclusive prefix of one int per thread over the block; total to *total.
__device__ __forceinline__ int block_excl_scan(int x, int *ws, int &total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    if (lane == 63) ws[wave] = incl;
    __syncthreads();
    int base = 0;
    total = 0;
#pragma unroll
    for (int i = 0; i < kBlock / 64; ++i) {
        const int c = ws[i];
        if (i < wave) base += c;
        total += c;
    }
    return base + incl - x;
}

// A hub chunk's partial (its pair terms and counts, summed over the block in a
// fixed tree order) goes to its slot (one thread); k_hub_sum adds the chunks of
// each hub in a fixed order once the score kernel is done.
__device__ void hub_chunk_store(const ScoreArgs &A, const double *red, const long long (*ired)[kBlock / 64],
                                int hub, int chunk) {
    HubPart hp;
    hp.raw = 0.0;
    hp.tI = hp.tII = 0;
    hp.pad = 0;
    for (int i = 0; i < kBlock / 64; ++i) {
        hp.raw += red[i];
        hp.tI += ired[0][i];
        hp.tII += ired[1][i];
    }
    A.hub_part[A.hub_first[hub] + chunk] = hp;
}

// A unit's type-I scan (below): the pairs with a non-empty out-list, in pair
// order per wavefront, the start bits of the items at hand, and the items that
// may close a triangle.
constexpr int kScanR = 2;             // work items per lane per round
constexpr int kScanSpan = 2048;       // items whose start bits are held at once
constexpr int kWaveHitCap = 192;      // candidates a wavefront holds before testing them
constexpr int kHitCap = kWaveHitCap * (kBlock / 64);
static_assert(kWaveHitCap >= 64 * kScanR, "a round's candidates always fit after a flush");
static_assert(kScanSpan % (64 * kScanR) == 0 && kScanSpan / 32 == 64, "whole rounds, one start word per lane");
struct OwnEnt {
    int delta;          // out-list start of the pair's w minus the pair's first item
    int pair;           // index in the unit
    unsigned int salt;  // the pair's part of the filter hash
    int pad;
};
struct TypeIShared {
    OwnEnt own[kBlock];                             // per wavefront: its non-empty pairs
    unsigned int start[kBlock / 64][kScanSpan / 32];
    double pW[kBlock];                              // w_w(C(u)) of each pair
};
// A candidate (item), later a hit, later the hit's two ordered triads.
union HitSlot {
    struct {
        int op;    // out-list position of v (the entry w -> v)
        int code;  // v; for a hit, where the edge test found (u, v)
    } c;
    double v;
};
struct HitBuf {
    HitSlot s[kHitCap];
    unsigned char p[kHitCap];  // pair (per wavefront: ascending)
};
static_assert(kBlock <= 256, "a pair index fits a byte");

// Lanes of one wavefront exchange data through LDS: the writes must be
// complete and visible before other lanes read them.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The exact edge test of a wavefront's held candidates [nt, nb) (from slot
// h0; the first nt are hits already): the hits move up, in order; returns the
// number of hits.
template <class Edge>
__device__ __forceinline__ int typeI_test(HitBuf &H, const Edge &edge, int h0, int nt, int nb, int lane) {
    for (int b0 = nt; b0 < nb; b0 += 64) {
        const int h = h0 + b0 + lane;
        int p = 0, op = 0, code = 0;
        bool hit = false;
        if (b0 + lane < nb) {
            p = H.p[h];
            op = H.s[h].c.op;
            hit = edge(p, H.s[h].c.code, code);
        }
        const unsigned long long m = __ballot(hit);
        wave_sync();
        if (hit) {
            const int s = h0 + nt + __popcll(m & ((1ull << lane) - 1ull));
            H.p[s] = (unsigned char)p;
            H.s[s].c.op = op;
            H.s[s].c.code = code;
        }
        nt += __popcll(m);
    }
    wave_sync();
    return nt;
}

// The terms of a wavefront's nb hits (from slot h0), then each pair's own lane
// adds its hits (a contiguous range of the list) in list order.
template <class Edge>
__device__ __forceinline__ void typeI_flush(const ScoreArgs &A, const TypeIShared &T, HitBuf &H, const Edge &edge,
                                            int h0, int nb, int lane, int me, bool mine, bool mem, double &val,
                                            int &t1) {
    for (int h = h0 + lane; h < h0 + nb; h += 64) {
        // the weights of the triangle {u, w, v}: w_v(C(u)), w_w(C(v)) and
        // w_v(C(w)), each the record at a leader slot (the out-list entry
        // w -> v holds the last two)
        const double W = T.pW[H.p[h]];
        const OutEnt e = A.oe[H.s[h].c.op];
        const double w_wv = A.prec[e.xy].w;
        const double w_vw = A.prec[e.yx].w;
        const double w_vu = edge.wvu(A, T, H.s[h].c.code, mem);
        H.s[h].v = cbrt(w_vu * w_wv * W) + cbrt(W * w_vw * w_vu);
    }
    wave_sync();
    if (mine) {
        int a = 0, b = nb;
        while (a < b) {
            const int mid = (a + b) >> 1;
            if ((int)H.p[h0 + mid] < me)
                a = mid + 1;
            else
                b = mid;
        }
        for (int h = a; h < nb && (int)H.p[h0 + h] == me; ++h) {
            val += H.s[h0 + h].v;
            t1 += 2;
        }
    }
    wave_sync();
}

// Type-I triads of a unit's pairs (Eq. RSI with v adjacent to u and C(v) !=
// C(u): the triangles of G').  The pair (u, w) finds the triangles {u, w, v}
// with v in out(w) (each triangle at u is found by exactly one of its two
// pairs).  Every position of every pair's out-list is one work item.  Each
// wavefront works through the items of its own 64 pairs, 64 items at a time
// (consecutive lanes read consecutive entries of one list, and no lane scans a
// long list alone), kScanR such groups with their loads in flight together;
// the wavefronts of the block do not wait for each other.  The kernel is bound
// by instructions issued and by the latency of the out-list reads (at n =
// 150 K, mean degree 71, 54 M items, half of the VALU's cycles), so an item
// takes few of both:
//   * its pair is found from one 64-bit word of start bits (a bit per item at
//     which a pair's list starts) by a count of the bits below the lane, where
//     a binary search of the pairs took six dependent LDS reads;
//   * a hashed filter of the unit's (u, v) pairs rejects nearly every
//     non-edge with one LDS read (the big hubs' filters are in memory), where
//     each item searched u's list; the few candidates are searched 64 at a
//     time.
// Candidates, and then hits, stay in item order, so each pair's hits are
// contiguous and in out-list order; every hit's two ordered triads (w, v) and
// (v, w),
//   cbrt(w_v(C(u)) w_w(C(v)) W) + cbrt(W w_v(C(w)) w_v(C(u))),  W = w_w(C(u)),
// are evaluated, one lane per hit, and the pair's own lane adds them to its
// sum, after the type-II terms, in list order (so the sum's order is fixed).
// `items` is the lane's out-list length (0 without a pair), `oo` its start and
// `salt` its part of the hash; the edge test's lists must be visible
// block-wide (a barrier) before the call.
//
// The pair's own facts are not needed before the hits are evaluated, so their
// loads are in flight during the scan: settle(), called once, waits for them
// and stores T.pW.  At the scan's end every wavefront passes one barrier of
// the block (kBlockW: hits read other wavefronts' T.pW), then evaluates its
// hits; a wavefront whose list fills up before evaluates what it holds at
// once, reading other wavefronts' weights from memory.
template <bool kBlockW, class Edge, class Settle>
__device__ __forceinline__ void typeI_scan(const ScoreArgs &A, TypeIShared &T, HitBuf &H, int items, int oo,
                                           unsigned int salt, const Edge &edge, const Settle &settle, double &val,
                                           int &t1) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int w0 = wave * 64;           // the wavefront's first pair
    const int h0 = wave * kWaveHitCap;  // and its candidate slots
    int incl = items;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    const int total = __builtin_amdgcn_readlane(incl, 63);
    const int first = incl - items;
    {
        const unsigned long long m = __ballot(items > 0);
        if (items > 0) {
            OwnEnt e;
            e.delta = oo - first;
            e.pair = tid;
            e.salt = salt;
            e.pad = 0;
            T.own[w0 + __popcll(m & ((1ull << lane) - 1ull))] = e;
        }
    }
    int nb = 0, nt = 0;  // held candidates of this wavefront, the first nt of them hits
    int seen = 0;        // pairs whose lists start before the group at hand
    int base = 0;
    bool settled = false;
    for (;;) {
        while (base < total && nb <= kWaveHitCap - 64 * kScanR) {
            const int sb = base & ~(kScanSpan - 1);
            if (base == sb) {  // the next span's start bits
                T.start[wave][lane] = 0u;
                wave_sync();
                if (items > 0 && first >= sb && first < sb + kScanSpan)
                    atomicOr(&T.start[wave][(first - sb) >> 5], 1u << ((first - sb) & 31));
                wave_sync();
            }
            int y[kScanR], op[kScanR], p[kScanR];
            unsigned int salts[kScanR];
#pragma unroll
            for (int r = 0; r < kScanR; ++r) {
                const int b = base + 64 * r;
                y[r] = -1;
                op[r] = p[r] = 0;
                salts[r] = 0u;
                if (b < total) {  // (uniform)
                    const unsigned int m0 = T.start[wave][(b - sb) >> 5], m1 = T.start[wave][((b - sb) >> 5) + 1];
                    const unsigned int lo = __builtin_amdgcn_readfirstlane((int)m0);
                    const unsigned int hi = __builtin_amdgcn_readfirstlane((int)m1);
                    const unsigned int mine = ((lane < 32 ? lo : hi) >> (lane & 31)) & 1u;
                    const int rank =
                        seen + (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u)) + (int)mine - 1;
                    seen += __popc(lo) + __popc(hi);
                    const OwnEnt e = T.own[w0 + rank];
                    p[r] = e.pair;
                    salts[r] = e.salt;
                    // (past the last item: the last one again, skipped below)
                    op[r] = e.delta + min(b + lane, total - 1);
                    y[r] = A.outl[op[r]];
                }
            }
#pragma unroll
            for (int r = 0; r < kScanR; ++r) {
                if (base + 64 * r >= total) break;
                const bool cand = base + 64 * r + lane < total && y[r] >= 0 && edge.maybe(salts[r], y[r]);
                const unsigned long long m = __ballot(cand);
                if (!m) continue;
                if (cand) {
                    const int s = h0 + nb + __popcll(m & ((1ull << lane) - 1ull));
                    H.p[s] = (unsigned char)p[r];
                    H.s[s].c.op = op[r];
                    H.s[s].c.code = y[r];
                }
                nb += __popcll(m);
            }
            base += 64 * kScanR;
        }
        const bool end = base >= total;
        wave_sync();
        nt = nb = typeI_test(H, edge, h0, nt, nb, lane);
        if (!end && nb <= kWaveHitCap - 64 * kScanR) continue;
        if (!settled) {
            settle();
            settled = true;
        }
        if (end && kBlockW)
            __syncthreads();  // once per wavefront
        else
            wave_sync();
        if (nb > 0) typeI_flush(A, T, H, edge, h0, nb, lane, tid, items > 0, !end, val, t1);
        if (end) return;
        nb = nt = 0;
    }
}

// Filter of a unit's (u, v) pairs in LDS: 256 pairs (an LDS hub: up to 1,024)
// in 16,384 bits, so 1.6 % (6 %) of the non-edges pass.
constexpr int kUnitFilterBits = 14;
constexpr int kUnitFilterWords = (1 << kUnitFilterBits) / 32;
__device__ __forceinline__ unsigned int unit_salt(int i) { return (unsigned int)i * 0x85EBCA6Bu; }
__device__ __forceinline__ unsigned int unit_hash(unsigned int salt, int y) {
    return ((unsigned int)y * 2654435761u + salt) >> (32 - kUnitFilterBits);
}
__device__ __forceinline__ void unit_filter_set(unsigned int *f, unsigned int salt, int y) {
    const unsigned int h = unit_hash(salt, y);
    atomicOr(&f[h >> 5], 1u << (h & 31));
}
__device__ __forceinline__ bool unit_filter_has(const unsigned int *f, unsigned int salt, int y) {
    const unsigned int h = unit_hash(salt, y);
    return (f[h >> 5] >> (h & 31)) & 1u;
}

// ------------------------------------------------------------ score units
// A score unit is either a tile -- <= kScoreTileV consecutive vertices with
// at most kScoreTileP foreign entries -- or one chunk of kScoreTileP pairs of
// a score hub whose foreign list fits in LDS.  Either way the foreign
// neighbours w of the unit's vertices are laid out in LDS (a vertex's
// entries ascending), one lane takes one pair (u, w), and the pair terms are
// summed in a fixed order: per vertex in pair order for a tile, in a tree
// over the chunk for a hub (k_hub_sum then adds a hub's chunk partials in a
// fixed order).
static_assert(kScoreTileV == kBlock && kScoreTileP == kBlock, "score unit size: one vertex and one pair per thread");

// A score unit's LDS: 27.5 KB would hold five workgroups on a CU, this form
// holds seven (a candidate takes nine bytes).
struct ScoreUnitShared {
    int w[kHubList];                 // foreign neighbours (a tile's at most kScoreTileP, an LDS hub's at most kHubList)
    unsigned short pb[kScoreTileV], pe[kScoreTileV];  // tile: pairs of each vertex
    unsigned char pu[kScoreTileP];                     // tile: vertex of each pair
    int ws[kBlock / 64];
    double red[kBlock / 64];
    long long ired[2][kBlock / 64];
    unsigned int filt[kUnitFilterWords];
    TypeIShared ti;
    union {  // three phases that never overlap
        int go[kScoreTileV];  // prologue: first slot of each of the tile's vertices
        HitBuf hits;          // type-I scan
        struct {              // epilogue: the lanes' pair terms
            double val;
            int t2, t1;
        } e[kBlock];
    } u;
};

// A hub chunk's partial: block tree sum of the lanes' terms (thread 0 gets it).
__device__ __forceinline__ void chunk_tree(double x, long long y1, long long y2, double *red,
                                           long long (*ired)[kBlock / 64]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        x += __shfl_xor(x, o);
        y1 += __shfl_xor(y1, o);
        y2 += __shfl_xor(y2, o);
    }
    if (lane == 0) {
        red[wave] = x;
        ired[0][wave] = y1;
        ired[1][wave] = y2;
    }
    __syncthreads();
}

// The edge test of a unit's type-I scan: u's foreign list is in LDS (a tile
// vertex's slice, or a hub's whole list, whose chunk's pairs are the list's
// positions [cbase, cbase + kBlock)).  It also gives a code for its hits, v's
// position, from which wvu() reads w_v(C(u)), the record of C(u) in v's list:
// it is the W of the pair (u, v), in T.pW when the unit has that pair, else
// (or with mem, where T.pW may not be whole) in memory.
struct UnitEdge {
    const ScoreUnitShared *S;
    int cbase;
    int slot0;          // slot of position 0
    const int32_t *vl;  // listed vertices (their slots are not consecutive), or null
    __device__ __forceinline__ bool maybe(unsigned int salt, int y) const { return unit_filter_has(S->filt, salt, y); }
    __device__ __forceinline__ bool operator()(int p, int y, int &code) const {
        const int i = S->pu[p], e = S->pe[i];
        const int k = lds_lower(S->w, S->pb[i], e, y);
        code = k;
        return k < e && S->w[k] == y;
    }
    __device__ __forceinline__ double wvu(const ScoreArgs &A, const TypeIShared &T, int code, bool mem) const {
        if (!mem && (unsigned int)(code - cbase) < (unsigned int)kBlock) return T.pW[code - cbase];
        int s = slot0 + code;
        if (vl) {
            const int i = S->pu[code];
            s = A.goff[vl[i]] + (code - S->pb[i]);
        }
        return A.prec[A.plink[s].lead].w;
    }
};

// vl: a unit of listed vertices vl[0, vn) (the incremental pass's rescored
// vertices) instead of the tile idx.
//
// A workgroup spends its time in a chain of dependent reads (some 20 us at n =
// 3 million, mean degree 30, with six of them on a CU), so the chain is kept
// short: a tile's lanes take its slots as they lie (a slot's vertex is a byte
// fixed with the schedule; slots that removals freed idle), so the links, the
// neighbours and the vertices' row facts are read together, and the pairs'
// records while the type-I scan runs.
__device__ void score_unit(const ScoreArgs &A, ScoreUnitShared &S, bool hub_unit, int idx, double wmax,
                           const int32_t *vl = nullptr, int vn = 0) {
    const int tid = threadIdx.x;
    for (int i = tid; i < kUnitFilterWords; i += kBlock) S.filt[i] = 0u;
    int v0 = 0, nv = 0, dp = 0, deg = 0, pb = 0;       // tile
    int hub = 0, chunk = 0, hu = 0, hdp = 0, hgo = 0;  // hub chunk
    int total = 0;                                     // hub chunk, listed vertices: pairs
    int slot = 0, s0 = 0, w = 0, own = 0;
    bool in = false, has = false;
    PairLink pl = {};
    if (hub_unit) {
        const int2 hc = A.hub_chunk[idx];
        hub = hc.x;
        chunk = hc.y;
        hu = A.hubs[hub];
        const VMeta m = A.meta[hu];
        hgo = A.goff[hu];
        hdp = m.deg - (m.q - m.p);  // <= the load-time count, which fits kHubList
        total = min(kBlock, max(0, hdp - chunk * kBlock));
        has = tid < total;
        if (has) {
            slot = hgo + chunk * kBlock + tid;
            pl = A.plink[slot];
        }
        __syncthreads();  // the cleared filter
        for (int j = tid; j < hdp; j += kBlock) {
            const int x = A.fcol[hgo + j];
            S.w[j] = x;
            unit_filter_set(S.filt, unit_salt(0), x);
        }
        S.pu[tid] = 0;  // one vertex, whose pairs are the whole list
        if (tid == 0) {
            S.pb[0] = 0;
            S.pe[0] = (unsigned short)hdp;
        }
        __syncthreads();
    } else {
        if (vl) {
            if (tid < vn) {
                const int v = vl[tid];
                const VMeta m = A.meta[v];
                deg = m.deg;
                dp = m.deg - (m.q - m.p);
                S.u.go[tid] = A.goff[v];
            }
            nv = vn;
            pb = block_excl_scan(dp, S.ws, total);  // (its barrier: the cleared filter)
            if (tid < nv)
                for (int q = pb; q < pb + dp; ++q) S.pu[q] = (unsigned char)tid;
            if (tid < nv) {
                S.pb[tid] = (unsigned short)pb;
                S.pe[tid] = (unsigned short)(pb + dp);
            }
            __syncthreads();
            in = tid < total;
            if (in) {
                own = S.pu[tid];
                slot = S.u.go[own] + (tid - S.pb[own]);
                pl = A.plink[slot];
                w = A.fcol[slot];
            }
        } else {
            const int2 tl = A.tiles[idx];
            v0 = tl.x;
            nv = tl.y - tl.x;
            const int s1 = A.goff[tl.y];
            s0 = A.goff[tl.x];
            in = tid < s1 - s0;
            if (in) {
                slot = s0 + tid;
                pl = A.plink[slot];
                w = A.fcol[slot];
                own = A.sown[slot];
            }
            if (tid < nv) {
                const VMeta m = A.meta[v0 + tid];
                pb = A.goff[v0 + tid] - s0;
                deg = m.deg;
                dp = m.deg - (m.q - m.p);
                S.pb[tid] = (unsigned short)pb;
                S.pe[tid] = (unsigned short)(pb + dp);
            }
            __syncthreads();  // the cleared filter
            if (in) S.pu[tid] = (unsigned char)own;
        }
        if (in) {
            has = tid < (int)S.pe[own];
            S.w[tid] = w;
            if (has) unit_filter_set(S.filt, unit_salt(own), w);
        }
        __syncthreads();
    }
    // ---- the lane's pair: its record is read while the type-I scan runs
    PairRec pr = {};
    if (has) pr = A.prec[pl.lead];
    const int items = has ? pl.on : 0;
    double val = 0.0;
    int t2 = 0, t1 = 0;
    auto settle = [&]() {
        if (has) {
            val = type2_pair(A, hub_unit ? hu : vl ? vl[own] : v0 + own, pr, pl);
            t2 = pr.f - 1;
            S.ti.pW[tid] = pr.w;
        }
    };
    // ---- type I (the candidate lists overlay the prologue's slots)
    UnitEdge E;
    E.S = &S;
    E.cbase = hub_unit ? chunk * kBlock : 0;
    E.slot0 = hub_unit ? hgo : s0;
    E.vl = vl;
    typeI_scan<true>(A, S.ti, S.u.hits, items, pl.oo, unit_salt(own), E, settle, val, t1);
    if (hub_unit) {
        chunk_tree(val, t1, t2, S.red, S.ired);
        if (tid == 0) hub_chunk_store(A, S.red, S.ired, hub, chunk);
        return;
    }
    // ---- epilogue: each vertex adds its pairs in order (the terms overlay the hit lists)
    __syncthreads();
    S.u.e[tid].val = val;
    S.u.e[tid].t2 = t2;
    S.u.e[tid].t1 = t1;
    __syncthreads();
    if (tid < nv && dp > 0) {
        double acc = 0.0;
        long long c1 = 0, c2 = 0;
#pragma unroll 4
        for (int q = pb; q < pb + dp; ++q) {
            acc += S.u.e[q].val;
            c2 += S.u.e[q].t2;
            c1 += S.u.e[q].t1;
        }
        score_store(A, vl ? vl[tid] : v0 + tid, deg, acc, c1, c2, wmax);
    }
}

// A hub whose foreign list exceeds kHubList: u's list stays in HBM.  The
// type-I edge test of (u, y) uses the out-lists instead: the edge is in
// exactly one of out(u) (staged in LDS when it fits) and out(y).
constexpr int kHubOutStage = 1024;
struct ScoreHubBigShared {
    double red[kBlock / 64];
    long long ired[2][kBlock / 64];
    int outu[kHubOutStage];
    TypeIShared ti;
    HitBuf hits;
};

// A big hub's neighbour filter: bit h(y) is set for every current foreign
// neighbour y of the hub (one multiplicative hash into 2^kFilterBits bits,
// built at the start of the score pass).  A clear bit proves that y is no
// neighbour; a set bit is checked exactly.
__device__ __forceinline__ uint32_t filter_hash(int y) {
    return ((uint32_t)y * 2654435761u) >> (32 - kFilterBits);
}

struct HubOutEdge {
    const int *stage;      // out(u) in LDS (n_stage entries), or null
    int n_stage;
    const int32_t *outl;
    const int64_t *oo;
    long long uo0, uo1;    // out(u) in HBM
    const uint32_t *filt;  // u's neighbour filter
    int u;
    __device__ __forceinline__ bool maybe(unsigned int, int y) const {
        const uint32_t h = filter_hash(y);
        return (filt[h >> 5] >> (h & 31)) & 1u;
    }
    // code: the out-list position of the edge, times two, plus 1 when it is
    // the entry v -> u (else u -> v)
    __device__ __forceinline__ bool operator()(int, int y, int &code) const {
        long long o = -1;
        if (stage) {
            const int k = lds_find_out(stage, n_stage, y);
            if (k >= 0) o = uo0 + k;
        } else {
            o = out_find(outl, uo0, uo1, y);
        }
        if (o >= 0) {
            code = (int)(o << 1);
            return true;
        }
        o = out_find(outl, oo[y], oo[y + 1], u);
        code = (int)(o << 1) | 1;
        return o >= 0;
    }
    __device__ __forceinline__ double wvu(const ScoreArgs &A, const TypeIShared &, int code, bool) const {
        const OutEnt e = A.oe[code >> 1];
        return A.prec[(code & 1) ? e.xy : e.yx].w;
    }
};

__device__ void score_hub_big(const ScoreArgs &A, ScoreHubBigShared &S, int hub, int chunk) {
    const int tid = threadIdx.x;
    const int u = A.hubs[hub];
    const VMeta m = A.meta[u];
    const int dp = m.deg - (m.q - m.p);
    const long long uo0 = A.oo[u], uo1 = A.oo[u + 1];
    const int n_out = (int)(uo1 - uo0);
    const bool staged = n_out <= kHubOutStage;
    if (staged)
        for (int j = tid; j < n_out; j += kBlock) S.outu[j] = A.outl[uo0 + j];
    const int k = chunk * kScoreTileP + tid;
    const bool has = k < dp;
    PairLink pl = {};
    PairRec pr = {};
    if (has) {
        pl = A.plink[A.goff[u] + k];
        pr = A.prec[pl.lead];
    }
    const int items = has ? pl.on : 0;
    double val = 0.0;
    int t2 = 0, t1 = 0;
    auto settle = [&]() {
        if (has) {
            val = type2_pair(A, u, pr, pl);
            t2 = pr.f - 1;
            S.ti.pW[tid] = pr.w;
        }
    };
    HubOutEdge E;
    E.stage = staged ? S.outu : nullptr;
    E.n_stage = n_out;
    E.outl = A.outl;
    E.oo = A.oo;
    E.uo0 = uo0;
    E.uo1 = uo1;
    E.filt = A.hfilter + (size_t)(hub - A.n_hubs_lds) * kFilterWords;
    E.u = u;
    __syncthreads();  // the staged out-list
    typeI_scan<false>(A, S.ti, S.hits, items, pl.oo, 0u, E, settle, val, t1);
    chunk_tree(val, t1, t2, S.red, S.ired);
    if (tid == 0) hub_chunk_store(A, S.red, S.ired, hub, chunk);
}

// Each big hub's neighbour filter from its current foreign list (after the
// row pass): built in LDS by one workgroup per hub, kFiltPer neighbours per
// thread loaded together, then written out whole.
constexpr int kFiltPer = 8;
__device__ __forceinline__ void build_filter(uint32_t *f, const VMeta *meta, const int32_t *goff, const int32_t *fcol,
                                             int hub, uint32_t *out) {
    for (int i = threadIdx.x; i < kFilterWords; i += kMidThreads) f[i] = 0u;
    const VMeta m = meta[hub];
    const int go = goff[hub];
    const int dp = m.deg - (m.q - m.p);
    __syncthreads();
    for (int j0 = threadIdx.x; j0 < dp; j0 += kFiltPer * kMidThreads) {
        int y[kFiltPer];
#pragma unroll
        for (int t = 0; t < kFiltPer; ++t) y[t] = fcol[go + min(j0 + t * kMidThreads, dp - 1)];  // (repeats set a bit again)
#pragma unroll
        for (int t = 0; t < kFiltPer; ++t) {
            const uint32_t x = filter_hash(y[t]);
            atomicOr(&f[x >> 5], 1u << (x & 31));
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kFilterWords; i += kMidThreads) out[i] = f[i];
}

// Type-II values by slot: for a run of w's list longer than one (the members
// of one community c adjacent to w), every member x gets
//   w_w(c)^(2/3) * (the sum of a_v over the run's other members v),
// the type-II terms of the pair (x, w) (Lemma 2), so the score pass reads one
// value where it would walk the run: a hub's run of hundreds of members is
// walked by each of its members, by one lane each, and at n = 3 million, mean
// degree 30, those walks (43 M gathers for 13.7 M pairs) held the score
// kernel at 2.0 ms.  Here each a_v is gathered once, into LDS, and a member
// sums the run from there, in run order (the order of type2_pair, so the bits
// are the same).  A workgroup takes kT2Tile consecutive slots and stages them
// with the rest of the runs cut at both ends; runs too long for the window
// are summed from memory.
constexpr int kT2Per = 2;
static_assert(kT2Tile == kT2Per * kMidThreads, "kT2Per slots per thread");
__device__ __forceinline__ void type2_tile(double *s_a, const PairRec *prec, const int32_t *fcol, const double *av,
                                           double *val2, int slots, int tile) {
    // (positions below are relative to the tile's first slot)
    prec += type2_first(tile);
    fcol += type2_first(tile);
    val2 += type2_first(tile);
    const int n = type2_count(slots, tile), tid = (int)threadIdx.x;
    // slots beyond a list that removals shrank hold the runs of an earlier
    // pass: their values are never read, and their runs stay in range
    PairRec rec[kT2Per];
    int lead[kT2Per], f[kT2Per];
#pragma unroll
    for (int j = 0; j < kT2Per; ++j) rec[j] = prec[min(tid + j * kMidThreads, n - 1)];
    const PairRec r0 = prec[0], r1 = prec[n - 1];
    const int l1 = r1.f < 0 ? n - 1 + r1.f : n - 1;
    const Type2Window w = type2_window(slots, tile, r0.f, l1, prec[l1].f);
    const int lo = w.lo, hi = w.hi;
#pragma unroll
    for (int j = 0; j < kT2Per; ++j) {
        const int s = tid + j * kMidThreads;
        lead[j] = rec[j].f < 0 ? s + rec[j].f : s;
        f[j] = s < n ? (rec[j].f < 0 ? prec[lead[j]].f : rec[j].f) : 0;
        if (f[j] > 1) s_a[s - lo] = av[fcol[s]];
    }
    for (int s = lo + tid; s < 0; s += kMidThreads) s_a[s - lo] = av[fcol[s]];
    for (int s = n + tid; s < hi; s += kMidThreads) s_a[s - lo] = av[fcol[s]];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kT2Per; ++j) {
        if (f[j] <= 1) continue;
        const int s = tid + j * kMidThreads;
        const int b = lead[j], e = lead[j] + f[j];
        double S = 0.0;
        if (b >= lo && e <= hi) {
            // (whole groups read consecutive doubles without a bound each: at n =
            // 3 million, mean degree 30, k_mid 135 -> 124 us)
            int i = b;
            for (; i + 8 <= e; i += 8) {
                double x[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) x[t] = s_a[i - lo + t];
#pragma unroll
                for (int t = 0; t < 8; ++t) S += i + t != s ? x[t] : 0.0;
            }
            for (; i < e; ++i) S += i != s ? s_a[i - lo] : 0.0;
        } else {
            for (int i = b; i < e; i += 8) {
                int y[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) y[t] = fcol[min(i + t, e - 1)];
                double x[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) x[t] = av[y[t]];
#pragma unroll
                for (int t = 0; t < 8; ++t) S += i + t < e && i + t != s ? x[t] : 0.0;
            }
        }
        const double c1 = cbrt(rec[j].w);
        val2[s] = c1 * c1 * S;
    }
}

// Everything between the row pass and the score pass, in one launch whose
// parts do not depend on each other: w_max (n_wmax workgroups), each graph's
// w_max of a batch (one wavefront per graph), the big hubs' filters (one
// workgroup each) and the type-II values (n_t2 tiles; 0 when the pairs sum
// their runs themselves).
struct MidArgs {
    const unsigned long long *wpart;
    int n_parts, n_wmax;
    unsigned long long *wblk;
    unsigned int *wticket;
    DevCounters *ctr;
    const int32_t *gblk_off, *gblk;
    int n_graphs;
    unsigned long long *gwmax;
    const int32_t *big_hubs;
    int n_filters;
    uint32_t *filters;
    const VMeta *meta;
    const int32_t *goff, *fcol;
    const PairRec *prec;
    const double *av;
    double *val2;
    int slots, n_t2;
};
constexpr int kMidGraphs = kMidThreads / 64;  // graphs per workgroup
// Two workgroups share a CU (64 registers; with 72, sixteen loads of a long run
// in flight, one did): n = 3 million, mean degree 30, 162 -> 137 us; n = 150,000,
// mean degree 71, 41 -> 34.
__global__ __launch_bounds__(kMidThreads, 8) void k_mid(MidArgs M) {
    __shared__ __align__(16) unsigned char buf[4 * kFilterWords];
    static_assert(sizeof(buf) == 8 * kT2Win, "a filter and a type-II window share the LDS");
    int b = (int)blockIdx.x;
    if (b < M.n_wmax) {
        reduce_wmax(M.wpart, M.n_parts, b, M.n_wmax, M.wblk, M.wticket, M.ctr);
        return;
    }
    b -= M.n_wmax;
    if (b < M.n_filters) {
        build_filter((uint32_t *)buf, M.meta, M.goff, M.fcol, M.big_hubs[b], M.filters + (size_t)b * kFilterWords);
        return;
    }
    b -= M.n_filters;
    if (b < M.n_t2) {
        type2_tile((double *)buf, M.prec, M.fcol, M.av, M.val2, M.slots, b);
        return;
    }
    b -= M.n_t2;
    const int gi = b * kMidGraphs + (int)(threadIdx.x >> 6);
    if (gi < M.n_graphs) reduce_wmax_graph(M.wpart, M.gblk_off, M.gblk, gi, M.gwmax);
}

union ScoreShared {
    ScoreUnitShared u;
    ScoreHubBigShared h;
};
// Six workgroups share a CU, with 80 registers, 10 of them spilled (44 bytes a
// lane): with registers for seven the compiler spills 33 of them (n = 3 million,
// mean degree 30: 1,413 against 1,362 us a pass; 128 graphs: 435 against 443).
static_assert(7 * sizeof(ScoreShared) <= 160 * 1024, "LDS for seven score workgroups per CU");

// Algorithm 1 Step 3 (Eq. RSI) for every border vertex, in one launch: the
// chunks of the hubs too large for LDS first (the longest units), then the
// LDS hubs' chunks, then the tiles (tile t of XCD x = t / per runs on a block
// of that XCD: blocks are dealt to the XCDs round-robin, so consecutive tiles
// share an L2).  Hub partials are summed by k_hub_sum.  Launches of their own
// for the hubs ended on one chunk's latency with nothing beside it.
__global__ __launch_bounds__(kBlock, 6) void k_score(ScoreArgs A) {
    __shared__ ScoreShared S;
    const int n_big = A.n_chunks - A.n_chunks_lds;
    const double wmax = bitsd(A.ctr->wmax_bits);
    int b = (int)blockIdx.x;
    if (b < n_big) {
        const int2 hc = A.hub_chunk[A.n_chunks_lds + b];
        score_hub_big(A, S.h, hc.x, hc.y);
        return;
    }
    b -= n_big;
    const bool hub_unit = b < A.n_chunks_lds;
    const int idx = hub_unit ? b : tile_of_block(b, A.n_chunks_lds, A.tiles_per_xcd);
    if (hub_unit || idx < A.n_tiles) score_unit(A, S.u, hub_unit, idx, wmax);
}

// The incremental pass's score work in one launch (the parts are
// independent and overlap): block i of a capped grid takes the work items
// i, i + gridDim.x, ... of one queue,
//   1. the listed big-hub chunks (all of them in a full pass),
//   2. the listed main blocks, LDS-hub chunks and tiles (all in a full pass),
//   3. the units of the affected tile vertices, largest bin first: 256 >> b
//      listed vertices of bin b per unit, so at most 256 pairs (none in a
//      full pass, whose tiles run whole).
// Every item runs as in the full launches; a unit's values are those of its
// vertices' tiles (a vertex's sum does not depend on the unit's others).
__global__ __launch_bounds__(kBlock) void k_score_inc(ScoreArgs A, const int32_t *big, const int32_t *main_,
                                                      const int32_t *abin, const unsigned long long *ictr,
                                                      uint8_t *hflag, int grid_rows, int grid_score, int grid_main) {
    __shared__ ScoreShared S;
    // the whole-hub flags of the marks were turned into lists: clear them
    for (int h = blockIdx.x * kBlock + threadIdx.x; h < A.n_hubs; h += gridDim.x * kBlock) hflag[h] = 0;
    const double wmax = bitsd(A.ctr->wmax_bits);
    const bool full = inc_full(ictr, grid_rows, grid_score);
    const long long n_big = full ? (long long)(A.n_chunks - A.n_chunks_lds) : (long long)ictr[kIcBig];
    const long long n_main = full ? (long long)grid_main : (long long)ictr[kIcMain];
    // units of bin b: ufirst[b] after the bins above b
    long long ufirst[kScoreBins], voff[kScoreBins], vcnt[kScoreBins], n_units = 0, off = 0;
#pragma unroll
    for (int b = 0; b < kScoreBins; ++b) {
        vcnt[b] = full ? 0 : (long long)ictr[kIcBins + b];
        voff[b] = off;
        off += vcnt[b];
    }
#pragma unroll
    for (int b = kScoreBins - 1; b >= 0; --b) {
        ufirst[b] = n_units;
        n_units += (vcnt[b] + (kBlock >> b) - 1) / (kBlock >> b);
    }
    const long long total = n_big + n_main + n_units;
    for (long long i = blockIdx.x; i < total; i += gridDim.x) {
        if (i < n_big) {
            const int c = full ? (int)i : big[i];
            const int2 hc = A.hub_chunk[A.n_chunks_lds + c];
            score_hub_big(A, S.h, hc.x, hc.y);
        } else if (i < n_big + n_main) {
            const long long j = i - n_big;
            const int bl = full ? (int)j : main_[j];
            const bool hub_unit = bl < A.n_chunks_lds;
            const int idx = hub_unit ? bl : tile_of_block(bl, A.n_chunks_lds, A.tiles_per_xcd);
            if (hub_unit || idx < A.n_tiles) score_unit(A, S.u, hub_unit, idx, wmax);
        } else {
            const long long u = i - n_big - n_main;
            int b = 0;  // units of bin b are [ufirst[b], ufirst[b - 1]); ufirst[kScoreBins - 1] = 0
            while (ufirst[b] > u) ++b;
            const int vpu = kBlock >> b;
            const long long start = voff[b] + (u - ufirst[b]) * vpu;
            const int nv = (int)min((long long)vpu, voff[b] + vcnt[b] - start);
            score_unit(A, S.u, false, -1, wmax, abin + start, nv);
        }
        __syncthreads();  // the next item's LDS
    }
}

// Each hub's score from its chunk partials (one wavefront per hub: lane l
// sums chunks l, l + 64, ... in order, then a fixed shuffle tree).  A hub
// whose foreign list became empty keeps the zeros the row pass wrote.
struct HubSumArgs {
    const int32_t *hubs, *hub_first;
    const HubPart *hub_part;
    int n_hubs;
    const VMeta *meta;
    const DevCounters *ctr;
    const unsigned long long *gwmax;
    const int32_t *vgraph;
    double *R, *raw;
    long long *tI, *tII;
};
__device__ __forceinline__ void hub_sum(const HubSumArgs &A) {
    const int hub = (int)blockIdx.x * (kBlock / 64) + (int)(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (hub >= A.n_hubs) return;
    const int first = A.hub_first[hub], nch = A.hub_first[hub + 1] - first;
    double acc = 0.0;
    long long c1 = 0, c2 = 0;
    for (int c = lane; c < nch; c += 64) {
        const HubPart q = A.hub_part[first + c];
        acc += q.raw;
        c1 += q.tI;
        c2 += q.tII;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        acc += __shfl_xor(acc, o);
        c1 += __shfl_xor(c1, o);
        c2 += __shfl_xor(c2, o);
    }
    if (lane == 0) {
        const int u = A.hubs[hub];
        const VMeta m = A.meta[u];
        if (m.deg - (m.q - m.p) > 0) {
            A.R[u] = score_value(acc, m.deg, bitsd(A.gwmax ? A.gwmax[A.vgraph[u]] : A.ctr->wmax_bits));
            A.raw[u] = acc;
            A.tI[u] = c1;
            A.tII[u] = c2;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_hub_sum(HubSumArgs A) { hub_sum(A); }

// The pass's triad totals from the per-vertex counts (read on demand: the
// incremental pass reruns vertices in units of its own, so per-workgroup
// partials of the full launch would go stale).
__global__ __launch_bounds__(1024) void k_reduce_score(const long long *tI, const long long *tII, long long n,
                                                       DevCounters *c) {
    __shared__ unsigned long long s[2][16];
    unsigned long long a = 0, b = 0;
    for (long long i = threadIdx.x; i < n; i += blockDim.x) {
        a += (unsigned long long)tI[i];
        b += (unsigned long long)tII[i];
    }
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o);
        b += __shfl_xor(b, o);
    }
    if ((threadIdx.x & 63) == 0) {
        s[0][threadIdx.x >> 6] = a;
        s[1][threadIdx.x >> 6] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long x = 0, y = 0;
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) {
            x += s[0][i];
            y += s[1][i];
        }
        c->sum_tI = x;
        c->sum_tII = y;
    }
}

// W1 = sum over G' pairs (u, w) of min(d'(u), d'(w)), the list elements a
// merge intersection would scan (reported for the algorithmic-byte count;
// computed when a reader asks, from the last pass's row facts).  One
// wavefront per vertex; per-block partials in wpart.
template <typename OffT>
__global__ __launch_bounds__(kBlock) void k_work_I(const OffT *off, const int32_t *col, const VMeta *meta, long long n,
                                                   unsigned long long *wpart) {
    __shared__ unsigned long long s[kBlock / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long acc = 0;
    for (long long x = (long long)blockIdx.x * (kBlock / 64) + wave; x < n; x += (long long)gridDim.x * (kBlock / 64)) {
        const VMeta m = meta[x];
        const int dpx = m.deg - (m.q - m.p);
        if (dpx == 0) continue;
        const OffT rb = off[x];
        for (int j = lane; j < m.deg; j += 64) {
            if (j >= m.p && j < m.q) continue;
            const VMeta my = meta[col[rb + j]];
            acc += (unsigned long long)min(dpx, my.deg - (my.q - my.p));
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (lane == 0) s[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int i = 0; i < kBlock / 64; ++i) t += s[i];
        wpart[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(kBlock) void k_reduce_work(const unsigned long long *wpart, DevCounters *c) {
    __shared__ unsigned long long s[kBlock / 64];
    unsigned long long t = 0;
    for (int i = threadIdx.x; i < kWorkBlocks; i += kBlock) t += wpart[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long z = 0;
        for (int i = 0; i < kBlock / 64; ++i) z += s[i];
        c->sum_workI = z;
    }
}

// ------------------------------------------------------------ link slots
// The link of the slot of (x, y): the leader of C(x)'s run and the slot of x
// in y's list, and y's out-list range.  Run at load; after removals k_mark_link
// rebuilds the links that moved.
// Lower bounds (first position holding an id >= key) of N keys, key i in the
// sorted row row[i][0, d[i]), found together: binary searches in lockstep,
// each step one independent load per key still searching.  DEC: removed
// entries (complemented in place, the row still ordered on the original
// ids) compare by their id.
template <int N, bool DEC>
__device__ __forceinline__ void lower_n(const int32_t *const *row, const int *d, const int *key, int *pos) {
    int lo[N], hi[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        lo[i] = 0;
        hi[i] = d[i];
    }
    for (;;) {
        bool more = false;
#pragma unroll
        for (int i = 0; i < N; ++i) more |= lo[i] < hi[i];
        if (!more) break;
        int mid[N], y[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            mid[i] = (lo[i] + hi[i]) >> 1;
            y[i] = lo[i] < hi[i] ? row[i][mid[i]] : 0;
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (lo[i] < hi[i]) {
                const int yi = DEC && y[i] < 0 ? ~y[i] : y[i];
                if (yi < key[i])
                    lo[i] = mid[i] + 1;
                else
                    hi[i] = mid[i];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) pos[i] = lo[i];
}

// ============================================================ load
// A graph's device form from the caller's CSR (large graphs; the host builds
// the small ones and those that fail a check here, to say what is wrong): the
// host renumbers the vertices, the device checks the rows, renumbers and sorts
// them, lists the foreign entries and orients G'.
// n = 200,000 with 3.7 M entries: rows 410 us, hub rows 75, symmetry 201, slots
// 34 + 66, all bound by the latency of dependent loads (5 in a row per vertex);
// load, pass, top-k and free in 3.9 ms, 26.7 with the host's build.

// Each caller id's internal id and community.
__global__ __launch_bounds__(kBlock) void k_load_map(const int32_t *new2old, const int32_t *lab, long long n,
                                                     int2 *map) {
    for (long long v = (long long)blockIdx.x * kBlock + threadIdx.x; v < n; v += (long long)gridDim.x * kBlock)
        map[new2old[v]] = make_int2((int)v, lab[v]);
}

// The rows of up to kLoadRow entries, one wavefront per row: check each entry
// (an id in range, no self-loop, the row ascending), renumber it, and write it
// at its rank among the row's new ids (counted: the ids are distinct, or the
// graph is refused).  An entry in a bad row is clamped, so everything stays in
// range; *bad tells.  Also each vertex's row length and foreign degree.
constexpr int kLoadRow = 1024;
template <typename OffIn, typename OffT>
__global__ __launch_bounds__(kBlock) void k_load_rows(const OffIn *off_in, const int32_t *col_in,
                                                      const int32_t *new2old, const int2 *map, long long n,
                                                      const OffT *off, int32_t *col, int32_t *clab, int32_t *deg,
                                                      int32_t *fgn, unsigned int *bad) {
    __shared__ __align__(16) int s_id[kBlock / 64][kLoadRow];
    int *ids = s_id[threadIdx.x >> 6];
    const int lane = threadIdx.x & 63;
    for (long long x = ((long long)blockIdx.x * kBlock + threadIdx.x) >> 6; x < n;
         x += ((long long)gridDim.x * kBlock) >> 6) {
        const int u = new2old[x];
        const long long b = (long long)off_in[u];
        const int d = (int)((long long)off_in[u + 1] - b);
        if (lane == 0) deg[x] = d;
        if (d > kLoadRow) continue;  // (k_load_hubs)
        const int cu = map[u].y;
        const long long o = (long long)off[x];
        unsigned int wrong = 0u;
        int foreign = 0;
        if (d <= 64) {
            int v = lane < d ? col_in[b + lane] : INT_MAX;
            const int prev = __shfl_up(v, 1);
            if (lane < d) {
                wrong = (v < 0 || v >= n || v == u || (lane > 0 && prev >= v)) ? 1u : 0u;
                v = min(max(v, 0), (int)(n - 1));
            }
            int2 m = make_int2(INT_MAX, cu);
            if (lane < d) m = map[v];
            int rank = 0;
            for (int j = 0; j < d; ++j) rank += __builtin_amdgcn_readlane(m.x, j) < m.x ? 1 : 0;
            if (lane < d) {
                col[o + rank] = m.x;
                clab[o + rank] = m.y;
            }
            foreign = __popcll(__ballot(m.y != cu));
        } else {
            for (int t = lane; t < ((d + 3) & ~3); t += 64) {
                int id = INT_MAX;  // (padding of the last four)
                if (t < d) {
                    int v = col_in[b + t];
                    if (v < 0 || v >= n || v == u || (t > 0 && col_in[b + t - 1] >= v)) wrong = 1u;
                    id = map[min(max(v, 0), (int)(n - 1))].x;
                }
                ids[t] = id;
            }
            wave_sync();
            for (int t0 = 0; t0 < d; t0 += 64) {
                const int t = t0 + lane;
                const int id = t < d ? ids[t] : INT_MAX;
                int rank = 0;
                for (int j = 0; j < d; j += 4) {
                    const int4 q = *(const int4 *)&ids[j];
                    rank += (q.x < id) + (q.y < id) + (q.z < id) + (q.w < id);
                }
                int c = cu;
                if (t < d) {
                    c = map[new2old[id]].y;
                    col[o + rank] = id;
                    clab[o + rank] = c;
                }
                foreign += __popcll(__ballot(c != cu));
            }
            wave_sync();  // the next row's ids
        }
        if (lane == 0) fgn[x] = foreign;
        if (__any(wrong != 0u) && lane == 0) atomicOr(bad, 1u);
    }
}

// A longer row, one workgroup each (hubs: internal ids): its new ids are set as
// bits of a range of 2^20 ids at a time and read back in order.
constexpr int kLoadBits = 1 << 20;
constexpr int kLoadWords = kLoadBits / 32 / 1024;  // words per thread
template <typename OffIn, typename OffT>
__global__ __launch_bounds__(1024) void k_load_hubs(const OffIn *off_in, const int32_t *col_in,
                                                    const int32_t *new2old, const int2 *map, const int32_t *lab,
                                                    long long n, const int32_t *hubs, const OffT *off, int32_t *col,
                                                    int32_t *clab, int32_t *fgn, unsigned int *bad) {
    __shared__ unsigned int s_bits[kLoadBits / 32];
    __shared__ int s_w[16], s_f;
    const int x = hubs[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int u = new2old[x], cu = lab[x];
    const long long b = (long long)off_in[u], o = (long long)off[x];
    const int d = (int)((long long)off_in[u + 1] - b);
    if (tid == 0) s_f = 0;
    int done = 0, foreign = 0;
    unsigned int wrong = 0u;
    for (long long r0 = 0; r0 < n; r0 += kLoadBits) {
        for (int i = tid; i < kLoadBits / 32; i += 1024) s_bits[i] = 0u;
        __syncthreads();
        for (int t = tid; t < d; t += 1024) {
            const int v = col_in[b + t];
            if (r0 == 0 && (v < 0 || v >= n || v == u || (t > 0 && col_in[b + t - 1] >= v))) wrong = 1u;
            const long long id = (long long)map[min(max(v, 0), (int)(n - 1))].x - r0;
            if (id >= 0 && id < kLoadBits) atomicOr(&s_bits[id >> 5], 1u << (id & 31));
        }
        __syncthreads();
        unsigned int w[kLoadWords];
        int cnt = 0;
#pragma unroll
        for (int j = 0; j < kLoadWords; ++j) {
            w[j] = s_bits[tid * kLoadWords + j];
            cnt += __popc(w[j]);
        }
        int incl = cnt;
#pragma unroll
        for (int q = 1; q < 64; q <<= 1) {
            const int y = __shfl_up(incl, q);
            if (lane >= q) incl += y;
        }
        if (lane == 63) s_w[wave] = incl;
        __syncthreads();
        int at = done + incl - cnt;
        for (int q = 0; q < 16; ++q) {
            if (q < wave) at += s_w[q];
            done += s_w[q];
        }
#pragma unroll
        for (int j = 0; j < kLoadWords; ++j) {
            for (unsigned int m = w[j]; m; m &= m - 1u) {
                const int id = (int)(r0 + 32ll * (tid * kLoadWords + j) + (__ffs((int)m) - 1));
                const int c = lab[id];
                col[o + at] = id;
                clab[o + at] = c;
                foreign += c != cu ? 1 : 0;
                ++at;
            }
        }
        __syncthreads();  // s_bits, s_w
    }
    // (a bad row may hold an id twice: the places left take its own id)
    for (int t = done + tid; t < d; t += 1024) {
        col[o + t] = x;
        clab[o + t] = cu;
    }
    if (foreign) atomicAdd(&s_f, foreign);
    if (wrong || (tid == 0 && done != d)) atomicOr(bad, 1u);
    __syncthreads();
    if (tid == 0) fgn[x] = s_f;
}

// Symmetry: every entry (x, y) has its (y, x).  A wavefront takes the rows of 64
// vertices, flattened over its lanes.  Not after a bad row (bit 0 of *bad, set
// by the launches before this one): places of its ids may be unwritten.
template <typename OffT>
__global__ __launch_bounds__(kBlock) void k_load_symmetric(const OffT *off, const int32_t *col, long long n,
                                                           unsigned int *bad) {
    __shared__ long long s_end[kBlock / 64][64];
    long long *end = s_end[threadIdx.x >> 6];
    const int lane = threadIdx.x & 63;
    if (*bad & 1u) return;
    for (long long v0 = (long long)blockIdx.x * kBlock + (threadIdx.x & ~63); v0 < n;
         v0 += (long long)gridDim.x * kBlock) {
        const long long first = (long long)off[v0], last = (long long)off[min(v0 + 64, n)];
        end[lane] = (long long)off[min(v0 + lane + 1, n)];
        wave_sync();
        unsigned int wrong = 0u;
        for (long long e = first + lane; e < last; e += 64) {
            int lo = 0, hi = 63;  // the row: the first whose end is beyond e
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (end[mid] > e)
                    hi = mid;
                else
                    lo = mid + 1;
            }
            const int x = (int)(v0 + lo);
            const int y = col[e];
            const long long yb = (long long)off[y];
            const int32_t *row[1] = {col + yb};
            const int d[1] = {(int)((long long)off[y + 1] - yb)};
            const int key[1] = {x};
            int p[1];
            lower_n<1, false>(row, d, key, p);
            if (p[0] >= d[0] || row[0][p[0]] != x) wrong = 1u;
        }
        if (__any(wrong != 0u) && lane == 0) atomicOr(bad, 2u);
        wave_sync();  // the next rows' ends
    }
}

// The foreign entries into their slots, in row order, and the number of those
// of higher rank (foreign degree, id) per vertex (count: out-list lengths), or,
// with oo, those entries into the out-lists.  One wavefront per row.
template <typename OffT>
__global__ __launch_bounds__(kBlock) void k_load_slots(const OffT *off, const int32_t *col, const int32_t *clab,
                                                       const int32_t *lab, const int32_t *goff, long long n,
                                                       int32_t *fcol, int32_t *count, const int64_t *oo,
                                                       int32_t *outl) {
    const int lane = threadIdx.x & 63;
    const unsigned long long lt = (1ull << lane) - 1ull;
    for (long long x = ((long long)blockIdx.x * kBlock + threadIdx.x) >> 6; x < n;
         x += ((long long)gridDim.x * kBlock) >> 6) {
        const int go = goff[x], f = goff[x + 1] - go;
        int higher = 0;
        if (!oo) {
            const long long b = (long long)off[x], e = (long long)off[x + 1];
            const int cx = lab[x];
            int at = go;
            for (long long j0 = b; j0 < e && at < go + f; j0 += 64) {
                const long long j = j0 + lane;
                const bool in = j < e && clab[j < e ? j : b] != cx;
                const int y = in ? col[j] : 0;
                const int g = in ? goff[y + 1] - goff[y] : 0;
                const unsigned long long m = __ballot(in);
                if (in) fcol[at + __popcll(m & lt)] = y;
                at += __popcll(m);
                higher += __popcll(__ballot(in && (g > f || (g == f && y > (int)x))));
            }
            if (lane == 0) count[x] = higher;
        } else {
            for (int j0 = 0; j0 < f; j0 += 64) {
                const bool in = j0 + lane < f;
                const int y = in ? fcol[go + j0 + lane] : 0;
                const int g = in ? goff[y + 1] - goff[y] : 0;
                const bool up = in && (g > f || (g == f && y > (int)x));
                const unsigned long long m = __ballot(up);
                if (up) outl[oo[x] + higher + __popcll(m & lt)] = y;
                higher += __popcll(m);
            }
        }
    }
}

// Exclusive prefix of n counts into out[0..n], in blocks of kPrefixBlock: the
// blocks' sums, their prefix by one workgroup, and each block's own.
constexpr int kPrefixBlock = 2048;
int prefix_blocks(int64_t n) { return (int)((n + kPrefixBlock - 1) / kPrefixBlock); }

__device__ __forceinline__ long long block_prefix(long long x, long long *ws, int waves, long long &total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    long long incl = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    if (lane == 63) ws[wave] = incl;
    __syncthreads();
    long long before = 0;
    total = 0;
    for (int w = 0; w < waves; ++w) {
        if (w < wave) before += ws[w];
        total += ws[w];
    }
    __syncthreads();
    return before + incl - x;
}

__global__ __launch_bounds__(kBlock) void k_prefix_sums(const int32_t *count, long long n, long long *sums) {
    __shared__ long long ws[kBlock / 64];
    long long s = 0, total;
    for (int j = 0; j < kPrefixBlock / kBlock; ++j) {
        const long long i = (long long)blockIdx.x * kPrefixBlock + j * kBlock + threadIdx.x;
        s += i < n ? count[i] : 0;
    }
    (void)block_prefix(s, ws, kBlock / 64, total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(1024) void k_prefix_top(long long *sums, int blocks) {
    __shared__ long long ws[16];
    long long base = 0;
    for (int i0 = 0; i0 < blocks; i0 += 1024) {
        const int i = i0 + (int)threadIdx.x;
        const long long x = i < blocks ? sums[i] : 0;
        long long total;
        const long long p = block_prefix(x, ws, 16, total);
        if (i < blocks) sums[i] = base + p;
        base += total;
    }
}

__global__ __launch_bounds__(kBlock) void k_prefix_out(const int32_t *count, long long n, const long long *sums,
                                                       int64_t *out) {
    __shared__ long long ws[kBlock / 64];
    long long base = sums[blockIdx.x];
    for (int j = 0; j < kPrefixBlock / kBlock; ++j) {
        const long long i = (long long)blockIdx.x * kPrefixBlock + j * kBlock + threadIdx.x;
        const long long x = i < n ? count[i] : 0;
        long long total;
        const long long p = block_prefix(x, ws, kBlock / 64, total);
        if (i < n) out[i] = base + p;
        if (i == n - 1) out[n] = base + p + x;
        base += total;
    }
}

template <typename OffIn, typename OffT>
static void load_rows_t(rs_graph *g, const LoadArgs &L) {
    DeviceGraph &D = g->d;
    const long long n = D.n;
    hipLaunchKernelGGL(k_load_map, dim3(grid_for(n, kBlock, 8192)), dim3(kBlock), 0, g->stream, D.new2old, D.lab, n,
                       L.map);
    hipLaunchKernelGGL((k_load_rows<OffIn, OffT>), dim3(grid_for(n, kBlock / 64, 16384)), dim3(kBlock), 0, g->stream,
                       (const OffIn *)L.off, L.col, D.new2old, L.map, n, (const OffT *)D.off, D.col, D.clab, D.deg,
                       L.fgn, L.bad);
    if (L.n_hubs > 0)
        hipLaunchKernelGGL((k_load_hubs<OffIn, OffT>), dim3(L.n_hubs), dim3(1024), 0, g->stream, (const OffIn *)L.off,
                           L.col, D.new2old, L.map, D.lab, n, L.hubs, (const OffT *)D.off, D.col, D.clab, L.fgn,
                           L.bad);
    hipLaunchKernelGGL(k_load_symmetric<OffT>, dim3(grid_for(n, kBlock, 8192)), dim3(kBlock), 0, g->stream,
                       (const OffT *)D.off, D.col, n, L.bad);
}

int load_hub_row() { return kLoadRow; }

rs_status launch_load_rows(rs_graph *g, const LoadArgs &L) {
    const bool w = L.offset_bytes == 8;
    if (g->d.off64)
        w ? load_rows_t<int64_t, long long>(g, L) : load_rows_t<int32_t, long long>(g, L);
    else
        w ? load_rows_t<int64_t, int32_t>(g, L) : load_rows_t<int32_t, int32_t>(g, L);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "row load launch");
}

template <typename OffT>
static void load_slots_t(rs_graph *g, int32_t *count, long long *sums) {
    DeviceGraph &D = g->d;
    const long long n = D.n;
    const int grid = grid_for(n, kBlock / 64, 16384), nb = prefix_blocks(n);
    hipLaunchKernelGGL(k_load_slots<OffT>, dim3(grid), dim3(kBlock), 0, g->stream, (const OffT *)D.off, D.col, D.clab,
                       D.lab, D.goff, n, D.fcol, count, (const int64_t *)nullptr, (int32_t *)nullptr);
    hipLaunchKernelGGL(k_prefix_sums, dim3(nb), dim3(kBlock), 0, g->stream, count, n, sums);
    hipLaunchKernelGGL(k_prefix_top, dim3(1), dim3(1024), 0, g->stream, sums, nb);
    hipLaunchKernelGGL(k_prefix_out, dim3(nb), dim3(kBlock), 0, g->stream, count, n, sums, D.oo);
    hipLaunchKernelGGL(k_load_slots<OffT>, dim3(grid), dim3(kBlock), 0, g->stream, (const OffT *)D.off, D.col, D.clab,
                       D.lab, D.goff, n, D.fcol, (int32_t *)nullptr, (const int64_t *)D.oo, D.outl);
}

rs_status launch_load_slots(rs_graph *g, int32_t *count, long long *sums) {
    if (g->d.off64)
        load_slots_t<long long>(g, count, sums);
    else
        load_slots_t<int32_t>(g, count, sums);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "slot load launch");
}

struct LinkArgs {
    const int32_t *lab, *cstart;
    const int32_t *goff, *fcol;
    const int64_t *oo;
    PairLink *plink;
    const int32_t *outl;        // out-lists (tombstones complemented)
    OutEnt *oe;                 // each out-list entry's leader slots
    const unsigned int *vmark;  // after removals: kRowChanged marks the rows that changed
    const VMeta *meta;          // after removals: the rows' facts (ell: the last pass's)
};

// The last x in [0, n) with off[x] <= s.
template <typename T>
__device__ __forceinline__ int owner_of(const T *off, long long n, long long s) {
    long long lo = 0, hi = n;
    while (hi - lo > 1) {
        const long long mid = (lo + hi) >> 1;
        if ((long long)off[mid] <= s)
            lo = mid;
        else
            hi = mid;
    }
    return (int)lo;
}

// Every slot's link (at load, when the lists are whole).  run_walk[0] gets
// the sum of the slots' distances to their leaders: half the steps in which
// the pairs would walk each other's runs.
__global__ __launch_bounds__(kBlock) void k_links(LinkArgs L, long long n, long long slots,
                                                  unsigned long long *run_walk) {
    unsigned long long walk = 0;
    for (long long s = (long long)blockIdx.x * kBlock + threadIdx.x; s < slots; s += (long long)gridDim.x * kBlock) {
        const int x = owner_of(L.goff, n, s);
        const int y = L.fcol[s];
        const int g0 = L.goff[y];
        const int32_t *rows[2] = {L.fcol + g0, L.fcol + g0};
        const int ds[2] = {L.goff[y + 1] - g0, L.goff[y + 1] - g0};
        const int keys[2] = {L.cstart[L.lab[x]], x};
        int k[2];
        lower_n<2, false>(rows, ds, keys, k);
        PairLink pl;
        pl.lead = g0 + k[0];
        pl.slot = g0 + k[1];
        pl.oo = (int)L.oo[y];
        pl.on = (int)(L.oo[y + 1] - L.oo[y]);
        L.plink[s] = pl;
        walk += (unsigned long long)(k[1] - k[0]);
    }
    __shared__ unsigned long long s_w[kBlock / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) walk += __shfl_xor(walk, o);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = walk;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kBlock / 64; ++i) walk += s_w[i];
        if (walk) atomicAdd(run_walk, walk);
    }
}

static LinkArgs link_args(rs_graph *g) {
    DeviceGraph &D = g->d;
    LinkArgs L;
    L.lab = D.lab;
    L.cstart = D.cstart;
    L.goff = D.goff;
    L.oo = D.oo;
    L.vmark = D.vmark;
    L.fcol = D.fcol;
    L.meta = D.meta;
    L.plink = D.plink;
    L.outl = D.outl;
    L.oe = D.oe;
    return L;
}

rs_status launch_links(rs_graph *g, unsigned long long *run_walk) {
    DeviceGraph &D = g->d;
    const long long slots = 2 * g->n_out;  // each G' edge has one out-list entry and two slots
    if (slots == 0) return RS_OK;
    hipLaunchKernelGGL(k_links, dim3(grid_for(slots, kBlock, 4096)), dim3(kBlock), 0, g->stream, link_args(g),
                       (long long)D.n, slots, run_walk);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "link-slot launch");
}

// The tile vertices' slots: each one's vertex, as its index in its score tile
// (with the schedule; a wavefront per tile vertex range).
__global__ __launch_bounds__(kBlock) void k_slot_owners(const int2 *tiles, int n_tiles, const int32_t *goff,
                                                        uint8_t *sown) {
    for (int t = (int)blockIdx.x; t < n_tiles; t += (int)gridDim.x) {
        const int2 tl = tiles[t];
        const int v = tl.x + (int)threadIdx.x;
        if (v < tl.y)
            for (int s = goff[v]; s < goff[v + 1]; ++s) sown[s] = (uint8_t)threadIdx.x;
    }
}

rs_status launch_slot_owners(rs_graph *g) {
    if (g->n_stiles == 0) return RS_OK;
    hipLaunchKernelGGL(k_slot_owners, dim3(std::min(g->n_stiles, 1 << 20)), dim3(kBlock), 0, g->stream, g->d.stiles,
                       g->n_stiles, g->d.goff, g->d.sown);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "slot owner launch");
}

// Each out-list entry x -> y (at load): the leader slots of C(y)'s run in x's
// list and of C(x)'s run in y's list; the owner x is the last with oo[x] <= o.
__global__ __launch_bounds__(kBlock) void k_out_entries(LinkArgs L, long long n, long long n_out) {
    for (long long o = (long long)blockIdx.x * kBlock + threadIdx.x; o < n_out; o += (long long)gridDim.x * kBlock) {
        const int x = owner_of(L.oo, n, o);
        const int y = out_id(L.outl[o]);
        const int xg = L.goff[x], yg = L.goff[y];
        const int32_t *rows[2] = {L.fcol + xg, L.fcol + yg};
        const int ds[2] = {L.goff[x + 1] - xg, L.goff[y + 1] - yg};
        const int keys[2] = {L.cstart[L.lab[y]], L.cstart[L.lab[x]]};
        int k[2];
        lower_n<2, false>(rows, ds, keys, k);
        OutEnt e;
        e.xy = xg + k[0];
        e.yx = yg + k[1];
        L.oe[o] = e;
    }
}

rs_status launch_out_entries(rs_graph *g) {
    DeviceGraph &D = g->d;
    const long long n_out = g->n_out;
    if (n_out == 0) return RS_OK;
    hipLaunchKernelGGL(k_out_entries, dim3(grid_for(n_out, kBlock, 65536)), dim3(kBlock), 0, g->stream, link_args(g),
                       (long long)D.n, n_out);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "out-entry launch");
}

// Each entry's neighbour community (once at load; compaction moves it with
// the entry): the row pass reads it in place of the id and its label.
__global__ __launch_bounds__(kBlock) void k_col_labels(const int32_t *col, const int32_t *lab, long long nnz,
                                                       int32_t *clab) {
    for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < nnz; e += (long long)gridDim.x * kBlock) {
        const int x = col[e];
        clab[e] = x >= 0 ? lab[x] : -1;
    }
}

rs_status launch_col_labels(rs_graph *g) {
    DeviceGraph &D = g->d;
    if (D.nnz == 0) return RS_OK;
    hipLaunchKernelGGL(k_col_labels, dim3(grid_for(D.nnz, kBlock, 65536)), dim3(kBlock), 0, g->stream, D.col, D.lab,
                       (long long)D.nnz, D.clab);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "entry label launch");
}


__global__ void k_zero_u64(unsigned long long *p, int count) {
    for (int i = threadIdx.x; i < count; i += blockDim.x) p[i] = 0ull;
}

// The end of an incremental pass: the hubs' sums (the first sum_blocks
// workgroups) and, when w_max changed, every other R recomputed from its raw
// sum (the same expression as the pass, so the bits equal a full pass's).
// Raw sums are 0 for vertices without foreign neighbours.
__global__ __launch_bounds__(kBlock) void k_inc_scores(HubSumArgs A, int sum_blocks, const int32_t *vscore,
                                                       const unsigned long long *wmax_old, long long n) {
    if ((int)blockIdx.x < sum_blocks) {
        hub_sum(A);
        return;
    }
    const unsigned long long wb = A.ctr->wmax_bits;
    if (wb == *wmax_old) return;
    const double wmax = bitsd(wb);
    for (long long u = (long long)((int)blockIdx.x - sum_blocks) * kBlock + threadIdx.x; u < n;
         u += (long long)((int)gridDim.x - sum_blocks) * kBlock) {
        if (vscore[u] < 0) continue;  // a hub
        const VMeta m = A.meta[u];
        A.R[u] = m.deg - (m.q - m.p) > 0 ? score_value(A.raw[u], m.deg, wmax) : 0.0;
    }
}

// ------------------------------------------------------------ pass launcher
// Workgroups of an incremental pass's launches (each loops over its list):
// enough to fill the chip, few enough that an empty list costs little.
constexpr int kIncGrid = 2048;

template <typename OffT>
static rs_status score_pass_t(rs_graph *g, bool inc) {
    DeviceGraph &D = g->d;
    hipEvent_t ev;
    RowArgs<OffT> A;
    A.off = (const OffT *)D.off;
    A.deg = D.deg;
    A.lab = D.lab;
    A.clab = D.clab;
    A.tables = (const TablesMem *)D.tables;
    A.tiles = D.rtiles;
    A.hubs = D.rhubs;
    A.n_tiles = g->n_rtiles;
    A.n_hubs = g->n_rhubs;
    A.tiles_per_xcd = (g->n_rtiles + 7) / 8;
    A.meta = D.meta;
    A.goff = D.goff;
    A.prec = D.prec;
    A.val2 = D.val2;
    A.blist = inc ? D.rlist : nullptr;
    A.wown = D.wown;
    A.av = D.av;
    A.R = D.R;
    A.raw = D.raw;
    A.tI = D.tI;
    A.tII = D.tII;
    A.part = D.part_rows;
    A.wmax_part = D.wmax_part;
    const int n_big = g->n_schunks - g->n_schunks_lds;
    const int grid_main = g->grid_score - n_big;
    if (inc) {
        timing_begin(g, K_ROWS, &ev);
        hipLaunchKernelGGL(k_rows_inc<OffT>, dim3(std::max(1, std::min(g->grid_rows, kIncGrid))), dim3(kBlock), 0,
                           g->stream, A, (const unsigned long long *)D.ictr, g->grid_rows, g->grid_score);
        timing_end(g, K_ROWS, ev);
    } else if (g->grid_rows > 0) {
        timing_begin(g, K_ROWS, &ev);
        hipLaunchKernelGGL(k_rows<OffT>, dim3(g->grid_rows), dim3(kBlock), 0, g->stream, A);
        timing_end(g, K_ROWS, ev);
    }
    const int n_big_hubs = g->n_shubs - g->n_shubs_lds;
    const long long slots = 2 * g->n_out;
    const bool by_slot = !inc && g->type2_by_slot;
    MidArgs M;
    M.wpart = D.wmax_part;
    M.n_parts = g->grid_rows;
    M.n_wmax = std::max(1, std::min(kWmaxBlocks, (g->grid_rows + 8191) / 8192));
    M.wblk = D.wblk;
    M.wticket = D.wticket;
    M.ctr = D.ctr;
    M.gblk_off = D.gblk_off;
    M.gblk = D.gblk;
    M.n_graphs = g->n_graphs;
    M.gwmax = D.gwmax;
    M.big_hubs = D.shubs + g->n_shubs_lds;
    M.n_filters = n_big_hubs;
    M.filters = D.hfilter;
    M.meta = D.meta;
    M.goff = D.goff;
    M.fcol = D.fcol;
    M.prec = D.prec;
    M.av = D.av;
    M.val2 = D.val2;
    M.slots = (int)slots;
    M.n_t2 = by_slot ? (int)((slots + kT2Tile - 1) / kT2Tile) : 0;
    timing_begin(g, K_MID, &ev);
    hipLaunchKernelGGL(k_mid, dim3(M.n_wmax + M.n_filters + M.n_t2 + (M.n_graphs + kMidGraphs - 1) / kMidGraphs),
                       dim3(kMidThreads), 0, g->stream, M);
    timing_end(g, K_MID, ev);

    ScoreArgs S;
    S.goff = D.goff;
    S.fcol = D.fcol;
    S.sown = D.sown;
    S.tiles = D.stiles;
    S.hubs = D.shubs;
    S.n_tiles = g->n_stiles;
    S.n_hubs = g->n_shubs;
    S.tiles_per_xcd = (g->n_stiles + 7) / 8;
    S.hub_first = D.shub_first;
    S.hub_chunk = D.shub_chunk;
    S.n_chunks = g->n_schunks;
    S.n_chunks_lds = g->n_schunks_lds;
    S.hub_part = D.hub_part;
    S.outl = D.outl;
    S.oo = D.oo;
    S.meta = D.meta;
    S.prec = D.prec;
    S.hfilter = D.hfilter;
    S.oe = D.oe;
    S.n_hubs_lds = g->n_shubs_lds;
    S.plink = D.plink;
    S.av = D.av;
    S.val2 = by_slot ? D.val2 : nullptr;
    S.R = D.R;
    S.raw = D.raw;
    S.gwmax = g->n_graphs > 0 ? D.gwmax : nullptr;
    S.vgraph = D.vgraph;
    S.tI = D.tI;
    S.tII = D.tII;
    S.ctr = D.ctr;
    const unsigned long long *ictr = D.ictr;
    if (inc) {
        timing_begin(g, K_SCORE, &ev);
        hipLaunchKernelGGL(k_score_inc, dim3(kIncGrid), dim3(kBlock), 0, g->stream, S, (const int32_t *)D.hlist,
                           (const int32_t *)D.slist, (const int32_t *)D.abin, ictr, D.hflag, g->grid_rows,
                           g->grid_score, grid_main);
        timing_end(g, K_SCORE, ev);
    } else {
        timing_begin(g, K_SCORE, &ev);
        if (g->grid_score > 0) hipLaunchKernelGGL(k_score, dim3(g->grid_score), dim3(kBlock), 0, g->stream, S);
        timing_end(g, K_SCORE, ev);
    }
    HubSumArgs U;
    U.hubs = D.shubs;
    U.hub_first = D.shub_first;
    U.hub_part = D.hub_part;
    U.n_hubs = g->n_shubs;
    U.meta = D.meta;
    U.ctr = D.ctr;
    U.gwmax = D.gwmax;
    U.vgraph = D.vgraph;
    U.R = D.R;
    U.raw = D.raw;
    U.tI = D.tI;
    U.tII = D.tII;
    const int sum_blocks = (g->n_shubs + kBlock / 64 - 1) / (kBlock / 64);
    const bool sums = sum_blocks > 0;
    if (sums) timing_begin(g, K_HUB_SUM, &ev);
    if (inc && D.n > 0)
        hipLaunchKernelGGL(k_inc_scores, dim3(sum_blocks + grid_for(D.n, kBlock, 4096)), dim3(kBlock), 0, g->stream, U,
                           sum_blocks, (const int32_t *)D.vscore, (const unsigned long long *)&D.ictr[kIcWmaxOld],
                           (long long)D.n);
    else if (sums)
        hipLaunchKernelGGL(k_hub_sum, dim3(sum_blocks), dim3(kBlock), 0, g->stream, U);
    if (sums) timing_end(g, K_HUB_SUM, ev);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "score pass launch");
    return RS_OK;
}

// (The few launches go straight to the stream: replaying them as a captured
// HIP graph started the first kernel later and cost 11 to 16 us a pass and
// top-k, 61 against 45 us at n = 2,000 and 243 against 232 at n = 1 million.)
rs_status launch_score_pass(rs_graph *g) {
    return g->d.off64 ? score_pass_t<long long>(g, false) : score_pass_t<int32_t>(g, false);
}

rs_status launch_score_incremental(rs_graph *g) {
    return g->d.off64 ? score_pass_t<long long>(g, true) : score_pass_t<int32_t>(g, true);
}

rs_status launch_reduce_counts(rs_graph *g) {
    DeviceGraph &D = g->d;
    hipLaunchKernelGGL(k_reduce_rows, dim3(1), dim3(kBlock), 0, g->stream, D.part_rows, g->grid_rows, D.ctr);
    hipLaunchKernelGGL(k_reduce_score, dim3(1), dim3(1024), 0, g->stream, D.tI, D.tII, (long long)D.n, D.ctr);
    if (D.off64)
        hipLaunchKernelGGL(k_work_I<long long>, dim3(kWorkBlocks), dim3(kBlock), 0, g->stream,
                           (const long long *)D.off, D.col, D.meta, (long long)D.n, D.wpart);
    else
        hipLaunchKernelGGL(k_work_I<int32_t>, dim3(kWorkBlocks), dim3(kBlock), 0, g->stream, (const int32_t *)D.off,
                           D.col, D.meta, (long long)D.n, D.wpart);
    hipLaunchKernelGGL(k_reduce_work, dim3(1), dim3(kBlock), 0, g->stream, D.wpart, D.ctr);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "reduce launch");
}

// ============================================================ top-k
__device__ __forceinline__ bool key_gt(const TopkKey &a, const TopkKey &b) {
    return a.hi > b.hi || (a.hi == b.hi && a.lo > b.lo);
}

__device__ __forceinline__ unsigned int key_digit(const TopkKey &k, int j) {
    switch (j) {
        case 0: return (unsigned int)(k.hi >> 48);
        case 1: return (unsigned int)(k.hi >> 32) & 0xffffu;
        case 2: return (unsigned int)(k.hi >> 16) & 0xffffu;
        case 3: return (unsigned int)k.hi & 0xffffu;
        case 4: return k.lo >> 16;
        default: return k.lo & 0xffffu;
    }
}

// A vertex's ranking key is (score bits, 0xffffffff - caller id), compared
// as one 96-bit number.  Scores are >= 0; the sign bit is cleared so that a
// -0.0 could never rank first.
__device__ __forceinline__ unsigned long long score_bits(double r) {
    return dbits(r) & 0x7fffffffffffffffull;
}

// Level-0 digit: the top 16 bits of the key (score bits only).
__device__ __forceinline__ unsigned int digit0_of(double r) { return (unsigned int)(score_bits(r) >> 48); }

// Level-0 bins: a score key's sign bit is clear, so its top 16 bits take
// values below 2^15.
constexpr int kHist0Bins = 32768;

// Level-0 histogram: each block (1024 threads) counts a contiguous chunk
// (< 2^16 keys) in an LDS histogram of 16-bit counters packed two per word
// (digit 0, which holds every zero score, is counted in registers), then adds
// its non-zero bins to the global histogram, and its sums of 256 consecutive
// bins to a 256-bin coarse histogram.  Few large blocks keep the number of
// global atomics (one per non-zero bin per block) small.
constexpr int kHistThreads = 1024;
constexpr int kHistPer = 16;  // keys per thread per step, loads all in flight together

// Global slot of level-0 bin b: consecutive bins 256 bytes apart (bin
// hi * 1024 + lo at lo * 64 + hi, a bijection of [0, 65536)).  Scores share
// their leading bits, so a pass fills a few hundred neighbouring bins, and
// every workgroup adds into all of them: spread over separate cache lines,
// those atomics no longer queue on a handful of lines.
__device__ __forceinline__ unsigned int hperm(unsigned int b) { return ((b & 1023u) << 6) | (b >> 10); }

// Loads of one step of a chunk scan [lo, hi) (hi > lo): kPer keys per thread,
// kThreads apart from v0.  Indexes past the chunk load its last key, which
// the caller skips, so no branch or select touches a loaded value before its
// use (either would wait for the load).  The flags are kept one per register:
// packed bytes would wait for their loads too.
template <int kPer, int kThreads>
__device__ __forceinline__ void load_keys(const double *R, const uint8_t *alive, long long v0, long long hi,
                                          double (&r)[kPer], unsigned int (&al)[kPer]) {
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const long long v = v0 + (long long)j * kThreads;
        const long long vc = v < hi ? v : hi - 1;
        r[j] = R[vc];
        al[j] = alive[vc];
    }
}

// Block 0 also resets the selection's list counters for the collect kernel.
__global__ __launch_bounds__(kHistThreads) void k_topk_hist(const double *R, const uint8_t *alive, long long n,
                                                            long long chunk, unsigned int *hist,
                                                            unsigned int *coarse, TopkState *st) {
    __shared__ uint4 sh4[kHist0Bins / 8];
    __shared__ unsigned int s_zero[kHistThreads / 64];
    unsigned int *sh = (unsigned int *)sh4;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->n_final = 0;
        st->n_tie = 0;
        st->overflow = 0;
    }
    const long long lo = (long long)blockIdx.x * chunk;
    const long long hi = min(n, lo + chunk);
    constexpr long long kStep = (long long)kHistPer * kHistThreads;
    const int steps = (int)((hi - lo + kStep - 1) / kStep);
    if (steps <= 0) return;  // (uniform; the grid never holds an empty chunk)
    unsigned int zeros = 0;
    for (int s = 0; s < steps; ++s) {
        const long long v0 = lo + (long long)s * kStep + threadIdx.x;
        double r[kHistPer];
        unsigned int al[kHistPer];
        load_keys<kHistPer, kHistThreads>(R, alive, v0, hi, r, al);
        if (s == 0) {  // clear the LDS histogram while the first loads are in flight
            for (int i = threadIdx.x; i < kHist0Bins / 8; i += kHistThreads) sh4[i] = make_uint4(0u, 0u, 0u, 0u);
            __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < kHistPer; ++j) {
            if (v0 + (long long)j * kHistThreads >= hi || !al[j]) continue;
            const unsigned int dig = digit0_of(r[j]);
            if (dig == 0u)
                ++zeros;
            else
                atomicAdd(&sh[dig >> 1], 1u << ((dig & 1u) * 16u));
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) zeros += __shfl_xor(zeros, o);
    if ((threadIdx.x & 63) == 0) s_zero[threadIdx.x >> 6] = zeros;
    __syncthreads();
    // flush: thread t takes the 16-byte words t, t + 1024, ... (8 bins each);
    // the 32 words of a coarse bin are 32 consecutive lanes of one wavefront,
    // whose sums a shuffle reduction adds.  Wavefronts whose words are all
    // zero (most: scores fill a few hundred bins) skip both.
    static_assert(kHist0Bins / 8 % kHistThreads == 0, "whole wavefronts per flush step");
    for (int i = threadIdx.x; i < kHist0Bins / 8; i += kHistThreads) {
        const uint4 x = sh4[i];
        unsigned int w[4] = {x.x, x.y, x.z, x.w};
        if (i == 0) {  // bin 0 (the low half of word 0) holds no LDS count: the zeros (< 2^16: the chunk is smaller)
            unsigned int z = 0;
            for (int q = 0; q < kHistThreads / 64; ++q) z += s_zero[q];
            w[0] += z;
        }
        unsigned int cs = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t) cs += (w[t] & 0xffffu) + (w[t] >> 16);
        if (!__any(cs != 0u)) continue;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (w[t] & 0xffffu) atomicAdd(&hist[hperm(8 * i + 2 * t)], w[t] & 0xffffu);
            if (w[t] >> 16) atomicAdd(&hist[hperm(8 * i + 2 * t + 1)], w[t] >> 16);
        }
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) cs += __shfl_xor(cs, o);
        if ((threadIdx.x & 31) == 0 && cs) atomicAdd(&coarse[i >> 5], cs);
    }
}

// The level-0 threshold, found by wavefront 0 of every block of the collect
// kernel from the finished histograms, with no barrier: lane l holds the
// positions 4l .. 4l + 3 of 256 counts in descending bin order.  wave_find
// returns, in every lane, the position where the running count reaches k,
// the count above it and the count at it (k <= the total; the caller checks).
struct Thresh0 {
    unsigned int bin;
    bool done;  // the bin is taken whole
};

__device__ __forceinline__ void wave_find(const long long (&c)[4], long long k, int &pos, long long &above,
                                          long long &at, long long &total) {
    const int lane = threadIdx.x & 63;
    const long long s = c[0] + c[1] + c[2] + c[3];
    long long incl = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    total = __shfl(incl, 63);
    const long long excl = incl - s;
    const unsigned long long m = __ballot(excl < k && k <= incl);
    const int L = m ? __ffsll((long long)m) - 1 : 0;
    long long a = __shfl(excl, L);
    long long q[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) q[j] = __shfl(c[j], L);
    int j = 0;
    while (j < 3 && a + q[j] < k) a += q[j++];
    pos = 4 * L + j;
    above = a;
    at = q[j];
}

// Wavefront 0 of a 1024-thread block: the coarse bin where the count from
// the top reaches k (cc: its lane's four coarse counts, loaded by the caller
// before anything else so that waiting for them waits for no later load),
// then the fine bin inside it.  Block 0 records the selection state for the
// later kernels.  Returns through LDS after one barrier of the whole block.
__device__ Thresh0 find_threshold0(const long long (&cc)[4], const unsigned int *hist, TopkState *st,
                                   long long k) {
    __shared__ Thresh0 s_res;
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        const bool publish = blockIdx.x == 0 && lane == 0;
        int pc;
        long long ac, mc, tot;
        wave_find(cc, k, pc, ac, mc, tot);
        Thresh0 res;
        if (tot < k) {  // cannot happen for k <= live keys: take all
            res.bin = 0u;
            res.done = true;
            if (publish) {
                st->k = k;
                st->digit = 0;
                st->thresh = 0;
                st->above = 0;
                st->take = 0;
                st->binsize = 0;
                st->done = 1u;
            }
        } else {
            const int c = 255 - pc;
            long long fc[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) fc[j] = hist[hperm((unsigned int)(256 * c + 255 - (4 * lane + j)))];
            int pf;
            long long af, mf, tf;
            wave_find(fc, k - ac, pf, af, mf, tf);
            const long long above = ac + af;
            res.bin = (unsigned int)(256 * c + 255 - pf);
            res.done = k == above + mf;
            if (publish) {
                st->k = k;
                st->digit = 0;
                st->thresh = res.bin;
                st->above = above;
                st->take = k - above;
                st->binsize = mf;
                st->done = res.done ? 1u : 0u;
            }
        }
        if (lane == 0) s_res = res;
    }
    __syncthreads();
    return s_res;
}

// Histogram of digit j over a key list (refinement of a large tie class).
// The refine levels are launched back to back with no host round trip: a
// level whose predecessor already took its threshold bin whole (done, at an
// earlier digit) does nothing.
__device__ __forceinline__ bool refine_finished(const TopkState *st, int level) {
    return st->done != 0u && (int)st->digit < level;
}

__global__ __launch_bounds__(kBlock) void k_list_hist(const TopkKey *list, const unsigned long long *count, int j,
                                                      const TopkState *st, unsigned int *hist) {
    __shared__ unsigned int s_d, s_c;  // the workgroup's aggregated digit and its count
    if (refine_finished(st, j)) return;
    const long long n = (long long)*count;
    if (threadIdx.x == 0) {
        s_d = 0xffffffffu;
        s_c = 0u;
    }
    __syncthreads();
    // keys of one wavefront that share a digit (common: a class of equal
    // scores shares every score digit, and ids share their high digits) are
    // added at once, into the workgroup's counter when the digit is the
    // workgroup's, so a class of equal keys costs one global atomic per
    // workgroup
    for (long long base = (long long)blockIdx.x * kBlock; base < n; base += (long long)gridDim.x * kBlock) {
        const long long i = base + threadIdx.x;
        const bool act = i < n;
        const unsigned int d = act ? key_digit(list[i], j) : 0u;
        const int lane = threadIdx.x & 63;
        unsigned long long pend = __ballot(act);
        // up to four digits shared by several lanes are added by one lane
        // each; the lanes left over add their own
        for (int r = 0; r < 4 && pend; ++r) {
            const int leader = __ffsll((long long)pend) - 1;
            const unsigned int dl = (unsigned int)__shfl((int)d, leader);
            const unsigned long long mm = __ballot(act && d == dl);
            if (lane == leader) {
                const unsigned int prev = atomicCAS(&s_d, 0xffffffffu, dl);
                if (prev == 0xffffffffu || prev == dl)
                    atomicAdd(&s_c, (unsigned int)__popcll(mm));
                else
                    atomicAdd(&hist[dl], (unsigned int)__popcll(mm));
            }
            pend &= ~mm;
        }
        if ((pend >> lane) & 1ull) atomicAdd(&hist[d], 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_c) atomicAdd(&hist[s_d], s_c);
}

// One block of 1024 threads: find the threshold digit of the current level,
// record it, and clear the histogram for the next use.  The bins are read as
// they lie (16 regions of 4,096, four bins a thread in each, coalesced); the
// region where the count from the top reaches `take` is found from the regions'
// sums, then the thread, then the bin.  With 64 consecutive bins a thread and a
// scan by doubling in LDS a level took 26 us, now 11.  (The 16 quads of bins
// take 96 registers and 32 bytes of scratch a lane.)
__global__ __launch_bounds__(1024) void k_topk_find(unsigned int *hist, TopkState *st, int level) {
    constexpr int kRegions = kTopkBins / 4096;
    __shared__ unsigned int s_w[kRegions][16];
    if (refine_finished(st, level)) return;  // (uniform; the histogram is still clear)
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const long long need = st->take;
    uint4 *h4 = (uint4 *)hist;
    uint4 x[kRegions];
#pragma unroll
    for (int i = 0; i < kRegions; ++i) x[i] = h4[i * 1024 + t];
#pragma unroll
    for (int i = 0; i < kRegions; ++i) h4[i * 1024 + t] = make_uint4(0u, 0u, 0u, 0u);
    // (a list holds at most n < 2^31 keys)
#pragma unroll
    for (int i = 0; i < kRegions; ++i) {
        const unsigned int s = wave_sum_last(x[i].x + x[i].y + x[i].z + x[i].w);
        if (lane == 63) s_w[i][wave] = s;
    }
    __syncthreads();
    // every thread walks the regions from the top, then the region's wavefronts
    long long above = 0;
    int reg = kRegions - 1, w = 15;
    for (; reg >= 0; --reg) {
        long long s = 0;
        for (int i = 0; i < 16; ++i) s += s_w[reg][i];
        if (above + s >= need) break;
        above += s;
    }
    if (reg < 0 || need <= 0) {  // cannot happen for need <= live keys: take all
        if (t == 0) {
            st->digit = (unsigned int)level;
            st->thresh = 0;
            st->take = 0;
            st->binsize = 0;
            st->done = 1u;
        }
        return;
    }
    for (; w > 0 && above + s_w[reg][w] < need; --w) above += s_w[reg][w];
    if (wave != w) return;
    uint4 b = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int i = 0; i < kRegions; ++i)
        if (i == reg) b = x[i];
    const unsigned int mine = b.x + b.y + b.z + b.w;
    unsigned int incl = mine;  // from this lane to the last: the counts of its bins and those above
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned int y = (unsigned int)__shfl_down((int)incl, o);
        if (lane + o < 64) incl += y;
    }
    const long long before = above + (incl - mine);
    if (before < need && need <= before + mine) {  // (one lane)
        const unsigned int c[4] = {b.x, b.y, b.z, b.w};
        long long cum = before;
        int i = 3;
        while (i > 0 && cum + c[i] < need) cum += c[i--];
        st->digit = (unsigned int)level;
        st->thresh = (unsigned int)(reg * 4096 + 4 * t + i);
        st->above += cum;
        st->take = need - cum;
        st->binsize = c[i];
        st->done = (need - cum == c[i]) ? 1u : 0u;
    }
}

// Block-aggregated append of the flagged threads' keys to list[*counter...].
__device__ __forceinline__ void block_push(TopkKey *list, unsigned long long *counter, bool act, const TopkKey &k,
                                           unsigned int *s_cnt, unsigned long long *s_base) {
    const unsigned long long m = __ballot(act);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) s_cnt[w] = (unsigned int)__popcll(m);
    __syncthreads();
    unsigned int before = 0, total = 0;
    for (int i = 0; i < kBlock / 64; ++i) {
        if (i < w) before += s_cnt[i];
        total += s_cnt[i];
    }
    if (threadIdx.x == 0 && total) *s_base = atomicAdd(counter, (unsigned long long)total);
    __syncthreads();
    if (act) list[*s_base + before + __popcll(m & ((1ull << __lane_id()) - 1ull))] = k;
    __syncthreads();
}

// Level-0 collect: keys above the threshold bin go to the final list, keys in
// it to the tie list.  Each block (1024 threads) issues its first loads, finds
// the threshold from the histograms while they are in flight, scans one
// contiguous chunk and stages its keys in LDS, then reserves room in each
// list with one atomic (keys beyond the staging capacity are reserved one by
// one).  The histograms are cleared by the ranking kernel that follows.
constexpr int kCollThreads = 1024;
constexpr int kCollPer = 8;       // keys per thread per step, loads all in flight together
constexpr int kCollStage = 2048;  // staged keys per list and block
__global__ __launch_bounds__(kCollThreads) void k_topk_collect(const double *R, const int32_t *new2old,
                                                               const uint8_t *alive, long long n, long long chunk,
                                                               long long k, const unsigned int *hist,
                                                               const unsigned int *coarse, TopkState *st,
                                                               TopkKey *fin, TopkKey *tie) {
    __shared__ TopkKey sf[kCollStage], stl[kCollStage];
    __shared__ unsigned int s_nf, s_nt;
    __shared__ unsigned long long s_bf, s_bt;
    if (threadIdx.x == 0) {
        s_nf = 0u;
        s_nt = 0u;
    }
    const long long lo = (long long)blockIdx.x * chunk;
    const long long hi = min(n, lo + chunk);
    constexpr long long kStep = (long long)kCollPer * kCollThreads;
    const int steps = (int)((hi - lo + kStep - 1) / kStep);
    if (steps <= 0) return;  // (uniform; the grid never holds an empty chunk, and block 0 starts at key 0)
    // the coarse counts first (wavefront 0 searches them; every lane loads
    // its four, no branch), then the first step's keys
    long long cc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) cc[j] = (long long)coarse[255 - (4 * (threadIdx.x & 63) + j)];
    double r[kCollPer];
    unsigned int al[kCollPer];
    load_keys<kCollPer, kCollThreads>(R, alive, lo + threadIdx.x, hi, r, al);
    __builtin_amdgcn_sched_barrier(0);  // no use of the loaded keys moves above the search
    const Thresh0 t0 = find_threshold0(cc, hist, st, k);
    const unsigned int th = t0.bin;
    const bool done = t0.done;
    for (int s = 0;;) {
        const long long v0 = lo + (long long)s * kStep + threadIdx.x;
#pragma unroll
        for (int j = 0; j < kCollPer; ++j) {
            if (v0 + (long long)j * kCollThreads >= hi || !al[j]) continue;
            const unsigned int dig = digit0_of(r[j]);
            const bool f = dig > th || (dig == th && done);
            const bool t = dig == th && !done;
            if (!f && !t) continue;
            const long long v = v0 + (long long)j * kCollThreads;
            TopkKey key;
            key.hi = score_bits(r[j]);
            key.lo = 0xffffffffu - (unsigned int)new2old[v];
            key.v = (int)v;
            const unsigned int i = atomicAdd(f ? &s_nf : &s_nt, 1u);
            if (i < (unsigned int)kCollStage)
                (f ? sf : stl)[i] = key;
            else if (f)
                fin[atomicAdd(&st->n_final, 1ull)] = key;
            else
                tie[atomicAdd(&st->n_tie, 1ull)] = key;
        }
        if (++s >= steps) break;
        load_keys<kCollPer, kCollThreads>(R, alive, lo + (long long)s * kStep + threadIdx.x, hi, r, al);
    }
    __syncthreads();
    const unsigned int cf = min(s_nf, (unsigned int)kCollStage), ct = min(s_nt, (unsigned int)kCollStage);
    if (threadIdx.x == 0) {
        if (cf) s_bf = atomicAdd(&st->n_final, (unsigned long long)cf);
        if (ct) s_bt = atomicAdd(&st->n_tie, (unsigned long long)ct);
    }
    __syncthreads();
    for (unsigned int i = threadIdx.x; i < cf; i += kCollThreads) fin[s_bf + i] = sf[i];
    for (unsigned int i = threadIdx.x; i < ct; i += kCollThreads) tie[s_bt + i] = stl[i];
}

// The tie class's largest score bits and the complement of its smallest (both
// zero before).
__global__ __launch_bounds__(kBlock) void k_tie_range(const TopkKey *tie, long long n, unsigned long long *range) {
    unsigned long long a = 0ull, b = 0ull;
    for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < n; i += (long long)gridDim.x * kBlock) {
        const unsigned long long h = tie[i].hi;
        a = max(a, h);
        b = max(b, ~h);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        a = max(a, (unsigned long long)__shfl_xor((long long)a, o));
        b = max(b, (unsigned long long)__shfl_xor((long long)b, o));
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&range[0], a);
        atomicMax(&range[1], b);
    }
}

// The list sizes of the refine levels from `first` on: the tie class's, then
// zeros.
__global__ void k_refine_counts(unsigned long long *cnt, int first, long long n_tie) {
    if ((int)threadIdx.x < 6) cnt[threadIdx.x] = (int)threadIdx.x == first - 1 ? (unsigned long long)n_tie : 0ull;
}

__global__ __launch_bounds__(kBlock) void k_list_collect(const TopkKey *list, const unsigned long long *count,
                                                         int level, TopkState *st, TopkKey *fin, TopkKey *tie,
                                                         unsigned long long *tie_count) {
    __shared__ unsigned int s_cnt[kBlock / 64];
    __shared__ unsigned long long s_base;
    if (refine_finished(st, level)) return;
    const long long n = (long long)*count;
    const int j = (int)st->digit;
    const unsigned int th = st->thresh;
    const bool done = st->done != 0u;
    for (long long base = (long long)blockIdx.x * kBlock; base < n; base += (long long)gridDim.x * kBlock) {
        const long long i = base + threadIdx.x;
        const bool act = i < n;
        TopkKey k;
        k.hi = 0;
        k.lo = 0;
        k.v = -1;
        unsigned int dig = 0;
        if (act) {
            k = list[i];
            dig = key_digit(k, j);
        }
        const bool to_final = act && (dig > th || (dig == th && done));
        const bool to_tie = act && dig == th && !done;
        if (__syncthreads_or(to_final)) block_push(fin, &st->n_final, to_final, k, s_cnt, &s_base);
        if (__syncthreads_or(to_tie)) block_push(tie, tie_count, to_tie, k, s_cnt, &s_base);
    }
}

// Final order of `count` keys (count <= kSortCap): bitonic sort, descending,
// in LDS by one block of 1024 threads.
__global__ __launch_bounds__(1024) void k_final_sort(const TopkKey *fin, long long count, const TopkState *st,
                                                     const double *R, const int32_t *new2old, int32_t *out_ids,
                                                     double *out_sc) {
    __shared__ TopkKey s[kSortCap];
    // the final list holds n_final keys, plus `take` ranked ties when the threshold bin was split
    const long long have = (long long)st->n_final + (st->done ? 0 : st->take);
    if (st->overflow || have != count) return;  // list incomplete: refinement pending
    int n2 = 1;
    while (n2 < count) n2 <<= 1;
    for (int i = threadIdx.x; i < n2; i += blockDim.x) {
        if (i < count) {
            s[i] = fin[i];
        } else {
            s[i].hi = 0;
            s[i].lo = 0;  // below every real key (a real key has lo >= 2^31)
            s[i].v = -1;
        }
    }
    __syncthreads();
    for (int k = 2; k <= n2; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < n2; i += blockDim.x) {
                const int l = i ^ j;
                if (l > i) {
                    const bool desc = (i & k) == 0;
                    const TopkKey x = s[i], y = s[l];
                    if (desc ? key_gt(y, x) : key_gt(x, y)) {
                        s[i] = y;
                        s[l] = x;
                    }
                }
            }
            __syncthreads();
        }
    }
    for (int i = threadIdx.x; i < count; i += blockDim.x) {
        out_ids[i] = new2old[s[i].v];
        out_sc[i] = R[s[i].v];
    }
}

// Final order of a longer list: each key's rank by pairwise comparison.
__global__ __launch_bounds__(kBlock) void k_final_rank(const TopkKey *fin, long long n, const TopkState *st,
                                                       const double *R, const int32_t *new2old, int32_t *out_ids,
                                                       double *out_sc) {
    __shared__ TopkKey tile[kBlock];
    const long long have = (long long)st->n_final + (st->done ? 0 : st->take);
    if (st->overflow || have != n) return;  // list incomplete: refinement pending
    for (long long base = (long long)blockIdx.x * kBlock; base < n; base += (long long)gridDim.x * kBlock) {
        const long long i = base + threadIdx.x;
        TopkKey me;
        me.hi = 0;
        me.lo = 0;
        me.v = -1;
        if (i < n) me = fin[i];
        long long rank = 0;
        for (long long t0 = 0; t0 < n; t0 += kBlock) {
            __syncthreads();
            if (t0 + threadIdx.x < n) tile[threadIdx.x] = fin[t0 + threadIdx.x];
            __syncthreads();
            const int lim = (int)min((long long)kBlock, n - t0);
            for (int jj = 0; jj < lim; ++jj) rank += key_gt(tile[jj], me) ? 1 : 0;
        }
        if (i < n) {
            out_ids[rank] = new2old[me.v];
            out_sc[rank] = R[me.v];
        }
    }
}

// ------------------------------------------------------------ rank by counting
// Ranking of a list of unique keys (the caller id is part of the key): a
// key's rank is the number of keys above it.  A workgroup of 1024 threads
// takes 64 keys (one per lane) and its 16 wavefronts each count over every
// 16th key of the list, staged in LDS tiles that every lane of a wavefront
// reads at the same place (broadcast); the 16 counts are summed.  Sixteen
// wavefronts per group keep enough of them on every CU to hide the LDS
// latency of the comparisons.
constexpr int kCountKeys = 64;
constexpr int kCountThreads = 1024;
constexpr int kCountSubs = kCountThreads / 64;
constexpr int kCountTile = 2048;
constexpr int kRankMax = 65536;  // longest list ranked here (final lists beyond: k_final_rank)

// 1 if the key (hi, lo) ranks above `me`, both halves compared without a
// branch: a short-circuit test waits for the score half's LDS read before
// issuing the id half's, which costs more than the extra read in the
// latency-bound ranking of a few thousand candidates (k_topk_rank).  The long
// lists of k_count_rank, bound by LDS issue instead, keep the short circuit.
__device__ __forceinline__ int key_above(unsigned long long hi, unsigned int lo, const TopkKey &me) {
    return (int)((hi > me.hi) | ((hi == me.hi) & (lo > me.lo)));
}

// The list a rank pass works on, and whether it is needed: the tie class of
// the threshold bin (mode 0, skipped when the bin was taken whole or is too
// large), or the final list of keff keys (mode 1, skipped while the list is
// incomplete).
__device__ __forceinline__ long long rank_count(const TopkState *st, int mode, long long keff) {
    if (mode == 0) {
        const long long n = (long long)st->n_tie;
        return (st->done || n > kTieCap) ? -1 : n;
    }
    const long long have = (long long)st->n_final + (st->done ? 0 : st->take);
    return (st->overflow || have != keff) ? -1 : keff;
}

// Mode 0: a tie key of rank r < take goes to the final list after the keys
// above the bin (a class too large to rank here is flagged for refinement
// digit by digit); mode 1: the key of rank r is the r-th output.
__global__ __launch_bounds__(kCountThreads) void k_count_rank(const TopkKey *list, TopkState *st, int mode,
                                                              long long keff, TopkKey *fin, const double *R,
                                                              const int32_t *new2old, int32_t *out_ids,
                                                              double *out_sc) {
    __shared__ unsigned long long s_hi[kCountTile];
    __shared__ unsigned int s_lo[kCountTile];
    __shared__ int s_part[kCountSubs][kCountKeys];
    const long long n = rank_count(st, mode, keff);
    if (mode == 0 && n < 0 && !st->done && blockIdx.x == 0 && threadIdx.x == 0) st->overflow = 1u;
    if (n < 0) return;
    const int lane = threadIdx.x & 63, sub = threadIdx.x >> 6;
    for (long long base = (long long)blockIdx.x * kCountKeys; base < n; base += (long long)gridDim.x * kCountKeys) {
        const long long i = base + lane;
        TopkKey me;
        me.hi = 0;
        me.lo = 0;
        me.v = -1;
        if (i < n) me = list[i];
        int cnt = 0;
        for (long long t0 = 0; t0 < n; t0 += kCountTile) {
            const int lim = (int)min((long long)kCountTile, n - t0);
            __syncthreads();  // the previous tile (and group) is done with LDS
            for (int j = threadIdx.x; j < lim; j += kCountThreads) {
                const TopkKey x = list[t0 + j];
                s_hi[j] = x.hi;
                s_lo[j] = x.lo;
            }
            __syncthreads();
#pragma unroll 8
            for (int j = sub; j < lim; j += kCountSubs)
                cnt += (s_hi[j] > me.hi || (s_hi[j] == me.hi && s_lo[j] > me.lo)) ? 1 : 0;
        }
        s_part[sub][lane] = cnt;
        __syncthreads();
        if (sub == 0 && i < n) {
            long long rank = 0;
#pragma unroll
            for (int q = 0; q < kCountSubs; ++q) rank += s_part[q][lane];
            if (mode == 0) {
                if (rank < st->take) fin[(long long)st->n_final + rank] = me;
            } else {
                out_ids[rank] = new2old[me.v];
                out_sc[rank] = R[me.v];
            }
        }
    }
}

// Common case: the final list and the threshold bin's keys together, at most
// `cap` candidates (the grid's 64 keys per workgroup), ordered by counting in
// the same layout as k_count_rank.  The final list's keys all lie above the
// bin's and keys are unique, so a candidate's place among all candidates is
// its place in the top-k; places below keff are written as ids and scores,
// recovered from the key (key = (score bits, 0xffffffff - caller id), scores
// >= +0), into the compact output block.  No selection inside the bin is
// needed.  flag = 1 when ranked here, 0 when the general path must run.
__global__ __launch_bounds__(kCountThreads) void k_topk_rank(const TopkState *st, const TopkKey *fin,
                                                             const TopkKey *tie, long long keff, long long cap,
                                                             int32_t *out_ids, double *out_sc, unsigned int *flag,
                                                             unsigned int *hist, unsigned int *coarse) {
    __shared__ unsigned long long s_hi[kCountTile];
    __shared__ unsigned int s_lo[kCountTile];
    __shared__ int s_part[kCountSubs][kCountKeys];
    // the level-0 histograms are no longer read: clear them for the next
    // call (and for the refinement levels of the general path)
    for (long long i = (long long)blockIdx.x * kCountThreads + threadIdx.x; i < kTopkBins / 4;
         i += (long long)gridDim.x * kCountThreads)
        ((uint4 *)hist)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (blockIdx.x == 0 && threadIdx.x < 256) coarse[threadIdx.x] = 0u;
    const long long nf = (long long)st->n_final;
    const long long n = nf + (st->done ? 0 : (long long)st->n_tie);
    const bool ok = n <= cap && n >= keff;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *flag = ok ? 1u : 0u;
        ((unsigned long long *)flag)[1] = (unsigned long long)(n - nf);  // the tie class
    }
    const long long base = (long long)blockIdx.x * kCountKeys;
    if (!ok || base >= n) return;  // uniform per workgroup
    const int lane = threadIdx.x & 63, sub = threadIdx.x >> 6;
    const long long i = base + lane;
    TopkKey me;
    me.hi = 0;
    me.lo = 0;
    me.v = -1;
    if (i < n) me = i < nf ? fin[i] : tie[i - nf];
    int cnt = 0;
    for (long long t0 = 0; t0 < n; t0 += kCountTile) {
        const int lim = (int)min((long long)kCountTile, n - t0);
        if (t0) __syncthreads();  // the previous tile is done with LDS
        for (int j = threadIdx.x; j < lim; j += kCountThreads) {
            const long long q = t0 + j;
            const TopkKey x = q < nf ? fin[q] : tie[q - nf];
            s_hi[j] = x.hi;
            s_lo[j] = x.lo;
        }
        __syncthreads();
#pragma unroll 8
        for (int j = sub; j < lim; j += kCountSubs) cnt += key_above(s_hi[j], s_lo[j], me);
    }
    s_part[sub][lane] = cnt;
    __syncthreads();
    if (sub == 0 && i < n) {
        long long rank = 0;
#pragma unroll
        for (int q = 0; q < kCountSubs; ++q) rank += s_part[q][lane];
        if (rank < keff) {
            out_ids[rank] = (int32_t)(0xffffffffu - me.lo);
            out_sc[rank] = __longlong_as_double((long long)me.hi);
        }
    }
}

// Candidates the common path ranks at most: the kSmallCap floor, or twice the
// requested count (the bin holding the k-th key rarely holds as many keys as
// lie above it), in whole workgroups.  Counting costs the square of the
// candidates, so beyond kUnionMax the general path (the threshold bin ranked
// alone, then the final list) is cheaper: 0, and the ranking kernel runs as
// one workgroup that only clears the histograms and sends the host there.
constexpr long long kUnionMax = 20480;
static long long rank_cap(long long keff) {
    long long cap = std::max<long long>(kSmallCap, 2 * keff);
    cap = (cap + kCountKeys - 1) / kCountKeys * kCountKeys;
    return cap <= kUnionMax ? cap : 0;
}

static rs_status final_order(rs_graph *g, long long keff) {
    DeviceGraph &D = g->d;
    hipEvent_t ev;
    timing_begin(g, K_TOPK_RANK, &ev);
    if (keff <= kSortCap) {
        hipLaunchKernelGGL(k_final_sort, dim3(1), dim3(1024), 0, g->stream, D.tfinal, keff, D.tstate, D.R,
                           D.new2old, D.tout_ids, D.tout_sc);
    } else if (keff <= kRankMax) {
        hipLaunchKernelGGL(k_count_rank, dim3((int)((keff + kCountKeys - 1) / kCountKeys)), dim3(kCountThreads), 0,
                           g->stream, (const TopkKey *)D.tfinal, D.tstate, 1, keff, (TopkKey *)nullptr, D.R,
                           D.new2old, D.tout_ids, D.tout_sc);
    } else {
        hipLaunchKernelGGL(k_final_rank, dim3(grid_for(keff, kBlock, 4096)), dim3(kBlock), 0, g->stream, D.tfinal,
                           keff, D.tstate, D.R, D.new2old, D.tout_ids, D.tout_sc);
    }
    timing_end(g, K_TOPK_RANK, ev);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "top-k order launch");
}

// The common path of top-k: the histogram, the collect (each block finds the
// threshold itself), and the ranking of the candidates by counting across
// workgroups into a compact device block [flag | ids | scores], copied once
// into pinned host memory.
static rs_status topk_common(rs_graph *g, long long keff) {
    DeviceGraph &D = g->d;
    hipEvent_t ev;
    long long chunk = (D.n + 63) / 64;  // about 64 blocks, each < 2^16 keys
    if (chunk < 16384) chunk = 16384;
    if (chunk > kHistChunk) chunk = kHistChunk;
    const int grid_h = (int)((D.n + chunk - 1) / chunk);
    timing_begin(g, K_TOPK_HIST, &ev);
    hipLaunchKernelGGL(k_topk_hist, dim3(grid_h), dim3(kHistThreads), 0, g->stream, D.R, D.alive, D.n, chunk,
                       D.thist, D.thist_c, D.tstate);
    timing_end(g, K_TOPK_HIST, ev);
    timing_begin(g, K_TOPK_COLLECT, &ev);
    long long cchunk = (D.n + 255) / 256;  // 64 to 256 blocks
    if (cchunk < 16384) cchunk = 16384;
    hipLaunchKernelGGL(k_topk_collect, dim3((int)((D.n + cchunk - 1) / cchunk)), dim3(kCollThreads), 0, g->stream,
                       D.R, D.new2old, D.alive, D.n, cchunk, keff, D.thist, D.thist_c, D.tstate, D.tfinal, D.ttie);
    timing_end(g, K_TOPK_COLLECT, ev);
    const size_t sc_off = 16 + ((4 * (size_t)keff + 7) & ~(size_t)7);
    char *dblk = D.tblk;
    const long long cap = rank_cap(keff);
    timing_begin(g, K_TOPK_RANK, &ev);
    hipLaunchKernelGGL(k_topk_rank, dim3((int)std::max<long long>(cap / kCountKeys, 1)), dim3(kCountThreads), 0,
                       g->stream, D.tstate, D.tfinal, D.ttie, keff, cap, (int32_t *)(dblk + 16),
                       (double *)(dblk + sc_off), (unsigned int *)dblk, D.thist, D.thist_c);
    timing_end(g, K_TOPK_RANK, ev);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(g->hpin, dblk, sc_off + 8 * (size_t)keff, hipMemcpyDeviceToHost, g->stream);
    return e == hipSuccess ? RS_OK : hip_fail(e, "top-k");
}

rs_status launch_topk(rs_graph *g, int64_t k, int32_t *ids, double *scores, int64_t *count) {
    DeviceGraph &D = g->d;
    const long long keff = k < g->n_alive ? k : g->n_alive;
    *count = keff;
    if (keff <= 0) return RS_OK;
    hipEvent_t ev;
    if (g->hpin_cap < keff) {
        void *p = nullptr;
        const hipError_t ea = hipHostMalloc(&p, 16 + 16 * (size_t)keff, hipHostMallocDefault);
        if (ea != hipSuccess) return hip_fail(ea, "pinned top-k buffer");
        if (g->hpin_own) (void)hipHostFree(g->hpin);
        g->hpin = p;
        g->hpin_cap = keff;
        g->hpin_own = true;
    }
    const size_t sc_off = 16 + ((4 * (size_t)keff + 7) & ~(size_t)7);
    rs_status cst = topk_common(g, keff);
    if (cst != RS_OK) return cst;
    hipError_t e = hipStreamSynchronize(g->stream);
    if (e != hipSuccess) return hip_fail(e, "top-k");
    if (*(const unsigned int *)g->hpin) {
        memcpy(ids, (const char *)g->hpin + 16, 4 * (size_t)keff);
        memcpy(scores, (const char *)g->hpin + sc_off, 8 * (size_t)keff);
        return RS_OK;
    }

    // General path: the tie class, by counting or digit by digit, then the
    // order of the final list (which already holds the keys above the class).
    const long long n_tie = (long long)((const unsigned long long *)g->hpin)[1];
    if (n_tie <= kTieCap) {
        timing_begin(g, K_TOPK_TIE, &ev);
        static_assert(kTieCap <= kRankMax, "a rankable tie class fits the counting ranker");
        hipLaunchKernelGGL(k_count_rank, dim3(kTieCap / kCountKeys), dim3(kCountThreads), 0, g->stream,
                           (const TopkKey *)D.ttie, D.tstate, 0, 0ll, D.tfinal, D.R, D.new2old, D.tout_ids, D.tout_sc);
        timing_end(g, K_TOPK_TIE, ev);
    } else {
        // A class larger than the pairwise ranker, as in a graph whose
        // removals leave most scores equal: then the score digits are skipped
        // and the ids' refined.  All levels are enqueued at once; the lists
        // only shrink, so the class bounds every level's grid, and the levels
        // after the one that finishes return at once.  (Three graphs of some
        // 40,000 to 70,000 vertices, six requests: 1,112 us with all levels at 16
        // keys a thread, the state read first and pageable copies; now 398.)
        unsigned long long *cnt = D.scratch_u;  // list sizes: [j] what level j leaves; [6], [7] the score range
        unsigned long long *range = (unsigned long long *)g->hpin;
        TopkKey *cur = D.ttie, *nxt = D.ttie2;
        const int grid_l = grid_for(n_tie, kBlock, 4096);
        const rs_status zst = launch_zero_u64(g, cnt + 6, 2);
        if (zst != RS_OK) return zst;
        hipLaunchKernelGGL(k_tie_range, dim3(grid_for(n_tie, 4 * kBlock, 256)), dim3(kBlock), 0, g->stream, cur, n_tie,
                           cnt + 6);
        e = hipMemcpyAsync(range, cnt + 6, 16, hipMemcpyDeviceToHost, g->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(g->stream);
        if (e != hipSuccess) return hip_fail(e, "top-k tie range");
        const int first = range[0] == ~range[1] ? 4 : 1;
        hipLaunchKernelGGL(k_refine_counts, dim3(1), dim3(64), 0, g->stream, cnt, first, n_tie);
        for (int j = first; j <= 5; ++j) {
            timing_begin(g, K_TOPK_FIND, &ev);
            hipLaunchKernelGGL(k_list_hist, dim3(grid_l), dim3(kBlock), 0, g->stream, cur, cnt + j - 1, j, D.tstate,
                               D.thist);
            hipLaunchKernelGGL(k_topk_find, dim3(1), dim3(1024), 0, g->stream, D.thist, D.tstate, j);
            timing_end(g, K_TOPK_FIND, ev);
            hipLaunchKernelGGL(k_list_collect, dim3(grid_l), dim3(kBlock), 0, g->stream, cur, cnt + j - 1, j, D.tstate,
                               D.tfinal, nxt, cnt + j);
            std::swap(cur, nxt);
        }
    }
    const rs_status rs_st = final_order(g, keff);
    if (rs_st != RS_OK) return rs_st;
    char *pin = (char *)g->hpin;
    e = hipMemcpyAsync(pin + 16, D.tout_ids, 4 * (size_t)keff, hipMemcpyDeviceToHost, g->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(pin + sc_off, D.tout_sc, 8 * (size_t)keff, hipMemcpyDeviceToHost, g->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(g->stream);
    if (e != hipSuccess) return hip_fail(e, "top-k copy");
    memcpy(ids, pin + 16, 4 * (size_t)keff);
    memcpy(scores, pin + sc_off, 8 * (size_t)keff);
    return RS_OK;
}

// ------------------------------------------------------------ batched top-k
// Top-k of every graph of a batch (k <= kBatchK), one wavefront per graph,
// the largest graphs first: each lane keeps the k best keys of its strided
// share of the graph's vertices, sorted, in its own LDS column (k * 64 keys
// per wavefront: lanes hit distinct banks and no barrier is needed).  Keys
// below a lower bound of the graph's k-th key are dropped with a register
// compare: first the k-th largest of the lanes' maximum keys (a first pass
// over the scores; k lanes hold a key at least that large), then, as lists
// fill, the largest k-th key over the lanes whose lists are full (that lane
// alone holds k keys at least as large).  The union of the lane
// lists holds the graph's top-k, which k rounds of a wavefront maximum over
// the list heads take out in order.  Scores are loaded kTopkGU per lane at a
// time so their latencies overlap.  Keys are (score bits, 0xffffffff - the
// caller's id within its graph); ids are distinct, so no two keys tie.
constexpr int kTopkGU = 16;

__device__ __forceinline__ bool key_gt(unsigned long long ah, unsigned int al, unsigned long long bh, unsigned int bl) {
    return ah > bh || (ah == bh && al > bl);
}

// Wavefront maximum of (flag, hi, lo) keys; lanes without a key pass flag 0.
__device__ __forceinline__ void wave_max_key(bool &f, unsigned long long &h, unsigned int &l, int &who) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long oh = (unsigned long long)__shfl_xor((long long)h, o);
        const unsigned int ol = (unsigned int)__shfl_xor((int)l, o);
        const int ow = __shfl_xor(who, o);
        const bool of = __shfl_xor((int)f, o) != 0;
        if (of && (!f || key_gt(oh, ol, h, l))) {
            h = oh;
            l = ol;
            who = ow;
            f = true;
        }
    }
}

__global__ __launch_bounds__(64) void k_topk_graphs(const double *R, const int32_t *new2old, const uint8_t *alive,
                                                    const int64_t *vstart, const int32_t *gorder, int n_graphs, int k,
                                                    int32_t *ids, double *scores, int64_t *counts) {
    extern __shared__ unsigned long long topk_lds[];  // [k][64] score bits, then [k][64] low keys
    unsigned long long *lhi = topk_lds;
    unsigned int *llo = (unsigned int *)(topk_lds + 64 * k);
    const int lane = threadIdx.x;
    for (int oi = blockIdx.x; oi < n_graphs; oi += gridDim.x) {
        const int gi = gorder[oi];
        const long long v0 = vstart[gi], v1 = vstart[gi + 1];
        // first pass: each lane's largest key, then the k-th largest of those
        bool mf = false;
        unsigned long long mh = 0;
        unsigned int ml = 0;
        for (long long base = v0; base < v1; base += 64 * kTopkGU) {
#pragma unroll
            for (int j = 0; j < kTopkGU; ++j) {
                const long long v = base + 64 * j + lane;
                if (v < v1 && alive[v]) {
                    const unsigned long long h = score_bits(R[v]);
                    const unsigned int l = 0xffffffffu - (unsigned int)(new2old[v] - (int)v0);
                    if (!mf || key_gt(h, l, mh, ml)) {
                        mh = h;
                        ml = l;
                        mf = true;
                    }
                }
            }
        }
        int rank = 0, nfull = 0;
        for (int m = 0; m < 64; ++m) {
            const unsigned long long oh = (unsigned long long)__shfl((long long)mh, m);
            const unsigned int ol = (unsigned int)__shfl((int)ml, m);
            const bool of = __shfl((int)mf, m) != 0;
            nfull += of;
            rank += of && key_gt(oh, ol, mh, ml);
        }
        const unsigned long long at_k = __ballot(mf && rank == k - 1);
        const bool have_lb = nfull >= k && at_k != 0ull;  // (uniform)
        unsigned long long lbh = 0;
        unsigned int lbl = 0;
        if (have_lb) {
            const int src = __ffsll((long long)at_k) - 1;
            lbh = (unsigned long long)__shfl((long long)mh, src);
            lbl = (unsigned int)__shfl((int)ml, src);
        }
        int cnt = 0;
        unsigned long long th = 0, tl_h = 0;  // wavefront bound; this lane's k-th key
        unsigned int tl = 0, tl_l = 0;
        bool have_th = false;
        for (long long base = v0; base < v1; base += 64 * kTopkGU) {
            unsigned long long hi[kTopkGU];
            unsigned int lo[kTopkGU];
            bool ok[kTopkGU];
#pragma unroll
            for (int j = 0; j < kTopkGU; ++j) {
                const long long v = base + 64 * j + lane;
                ok[j] = v < v1;
                hi[j] = 0;
                lo[j] = 0;
                if (ok[j]) {
                    ok[j] = alive[v] != 0;
                    hi[j] = score_bits(R[v]);
                    lo[j] = 0xffffffffu - (unsigned int)(new2old[v] - (int)v0);
                }
            }
#pragma unroll
            for (int j = 0; j < kTopkGU; ++j) {
                if (!ok[j]) continue;
                if (have_lb && key_gt(lbh, lbl, hi[j], lo[j])) continue;
                if (have_th && !key_gt(hi[j], lo[j], th, tl)) continue;
                if (cnt == k && !key_gt(hi[j], lo[j], tl_h, tl_l)) continue;
                int p = cnt < k ? cnt++ : k - 1;
                while (p > 0 && key_gt(hi[j], lo[j], lhi[64 * (p - 1) + lane], llo[64 * (p - 1) + lane])) {
                    lhi[64 * p + lane] = lhi[64 * (p - 1) + lane];
                    llo[64 * p + lane] = llo[64 * (p - 1) + lane];
                    --p;
                }
                lhi[64 * p + lane] = hi[j];
                llo[64 * p + lane] = lo[j];
                if (cnt == k) {
                    tl_h = lhi[64 * (k - 1) + lane];
                    tl_l = llo[64 * (k - 1) + lane];
                }
            }
            bool f = cnt == k;
            unsigned long long h = f ? tl_h : 0ull;
            unsigned int l = f ? tl_l : 0u;
            int who = lane;
            wave_max_key(f, h, l, who);
            if (f) {
                have_th = true;
                th = h;
                tl = l;
            }
        }
        int ptr = 0, taken = 0;
        for (int r = 0; r < k; ++r) {
            bool f = ptr < cnt;
            unsigned long long hh = f ? lhi[64 * ptr + lane] : 0ull;
            unsigned int hl = f ? llo[64 * ptr + lane] : 0u;
            int who = lane;
            wave_max_key(f, hh, hl, who);
            if (!f) break;  // fewer live vertices than k (uniform across the wavefront)
            if (lane == who) ++ptr;
            if (lane == 0) {
                ids[(long long)gi * k + r] = (int32_t)(0xffffffffu - hl);
                scores[(long long)gi * k + r] = __longlong_as_double((long long)hh);
            }
            ++taken;
        }
        if (lane == 0) counts[gi] = taken;
    }
}

// Segmented form, for batches whose graphs have at most 64 segments of
// kSegKeys = 64 * kTopkGU vertices: one wavefront per segment holds its keys
// in registers (kTopkGU per lane) and takes out the segment's top-k; one
// wavefront per graph merges the lists of a graph of several segments.  Both
// find a key that at least k keys reach, keep the keys that reach it (some k
// to 2k of them) and place each by counting the larger ones: keys are unique.
// (k rounds of a wavefront maximum took a segment 23 us for k = 7 and 57 us for
// k = 20; the placing takes one pass whatever k is.)
constexpr int kSegKeys = 64 * kTopkGU;
static_assert(kSegKeys == kSegVerts, "a segment is one key per lane and register slot");
constexpr int kSegCand = kTopkGU * kBatchK;  // candidates: the keys of at most k lanes

__device__ __forceinline__ unsigned long long lane_u64(unsigned long long x, int l) {
    return ((unsigned long long)(unsigned int)__builtin_amdgcn_readlane((int)(x >> 32), l) << 32) |
           (unsigned int)__builtin_amdgcn_readlane((int)x, l);
}

// The k-th largest of the lanes' keys (f: the lane has one); false when fewer
// than k lanes have keys.
__device__ __forceinline__ bool lane_kth(bool f, unsigned long long h, unsigned int l, int k, unsigned long long &kh,
                                         unsigned int &kl) {
    const unsigned long long full = __ballot(f);
    if (__popcll(full) < k) return false;
    int rank = 0;
    for (unsigned long long m = full; m; m &= m - 1ull) {
        const int s = __ffsll((long long)m) - 1;
        rank += key_gt(lane_u64(h, s), (unsigned int)__builtin_amdgcn_readlane((int)l, s), h, l) ? 1 : 0;
    }
    const unsigned long long at = __ballot(f && rank == k - 1);  // (one lane: keys are unique)
    const int s = __ffsll((long long)at) - 1;
    kh = lane_u64(h, s);
    kl = (unsigned int)__builtin_amdgcn_readlane((int)l, s);
    return true;
}

// Place the n candidates of a wavefront's list: emit(rank, hi, lo) for the k
// largest.
template <class Emit>
__device__ __forceinline__ void place_candidates(const unsigned long long *ch, const unsigned int *cl, int n, int k,
                                                 const Emit &emit) {
    for (int i = threadIdx.x & 63; i < n; i += 64) {
        const unsigned long long h = ch[i];
        const unsigned int l = cl[i];
        int rank = 0;
        int t = 0;
        for (; t + 8 <= n; t += 8) {  // eight reads in flight together
            unsigned long long th[8];
            unsigned int tl[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                th[j] = ch[t + j];
                tl[j] = cl[t + j];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) rank += key_gt(th[j], tl[j], h, l) ? 1 : 0;
        }
        for (; t < n; ++t) rank += key_gt(ch[t], cl[t], h, l) ? 1 : 0;
        if (rank < k) emit(rank, h, l);
    }
}

__global__ __launch_bounds__(kBlock) void k_topk_seg(const double *R, const int32_t *new2old, const uint8_t *alive,
                                                     const int64_t *vstart, const int32_t *seg_g,
                                                     const int32_t *sfirst, int n_segs, int k,
                                                     unsigned long long *c_hi, unsigned int *c_lo, int32_t *c_cnt,
                                                     int32_t *ids, double *scores, int64_t *counts) {
    __shared__ unsigned long long s_h[kBlock / 64][kSegCand];
    __shared__ unsigned int s_l[kBlock / 64][kSegCand];
    const int seg = (int)blockIdx.x * (kBlock / 64) + (int)(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (seg >= n_segs) return;  // whole wavefronts leave; no barrier follows
    unsigned long long *ch = s_h[threadIdx.x >> 6];
    unsigned int *cl = s_l[threadIdx.x >> 6];
    const int gi = seg_g[seg];
    const int sf = sfirst[gi];
    const bool whole = sfirst[gi + 1] - sf == 1;  // the graph's only segment: its lists are the graph's
    const long long gv0 = vstart[gi];
    const long long s0 = gv0 + (long long)(seg - sf) * kSegKeys;
    const long long s1 = min(s0 + (long long)kSegKeys, (long long)vstart[gi + 1]);
    unsigned long long hi[kTopkGU], bh = 0ull;
    unsigned int lo[kTopkGU], bl = 0u;
    unsigned int valid = 0u;
    if (s1 > s0) {
        double sc[kTopkGU];
        unsigned int al[kTopkGU], id[kTopkGU];
#pragma unroll
        for (int j = 0; j < kTopkGU; ++j) {  // (slots past the segment load its last vertex, and are skipped)
            const long long v = min(s0 + 64 * j + lane, s1 - 1);
            sc[j] = R[v];
            al[j] = alive[v];
            id[j] = (unsigned int)new2old[v];
        }
#pragma unroll
        for (int j = 0; j < kTopkGU; ++j) {
            hi[j] = score_bits(sc[j]);
            lo[j] = 0xffffffffu - (id[j] - (unsigned int)gv0);
            const bool ok = s0 + 64 * j + lane < s1 && al[j];
            valid |= (ok ? 1u : 0u) << j;
            if (ok && ((valid & ((1u << j) - 1u)) == 0u || key_gt(hi[j], lo[j], bh, bl))) {
                bh = hi[j];
                bl = lo[j];
            }
        }
    }
    unsigned long long kh = 0ull;
    unsigned int kl = 0u;
    const bool bound = lane_kth(valid != 0u, bh, bl, k, kh, kl);
    int n = 0;  // at most kTopkGU * k: a lane with a candidate is one of the k, or there are fewer than k lanes
#pragma unroll
    for (int j = 0; j < kTopkGU; ++j) {
        const bool c = ((valid >> j) & 1u) && !(bound && key_gt(kh, kl, hi[j], lo[j]));
        const unsigned long long m = __ballot(c);
        if (c) {
            const int i = n + __popcll(m & ((1ull << lane) - 1ull));
            ch[i] = hi[j];
            cl[i] = lo[j];
        }
        n += __popcll(m);
    }
    wave_sync();
    place_candidates(ch, cl, n, k, [&](int rank, unsigned long long h, unsigned int l) {
        if (whole) {
            ids[(long long)gi * k + rank] = (int32_t)(0xffffffffu - l);
            scores[(long long)gi * k + rank] = __longlong_as_double((long long)h);
        } else {
            c_hi[(long long)seg * k + rank] = h;
            c_lo[(long long)seg * k + rank] = l;
        }
    });
    if (lane == 0) {
        if (whole)
            counts[gi] = min(n, k);
        else
            c_cnt[seg] = min(n, k);
    }
}

constexpr int kMergePer = 8;  // keys per lane per step, loads in flight together
__global__ __launch_bounds__(64) void k_topk_merge(const unsigned long long *c_hi, const unsigned int *c_lo,
                                                   const int32_t *c_cnt, const int32_t *sfirst, int n_graphs, int k,
                                                   int32_t *ids, double *scores, int64_t *counts) {
    extern __shared__ unsigned long long topk_lds[];  // [64 k] score bits, then [64 k] low keys
    unsigned long long *ch = topk_lds;
    unsigned int *cl = (unsigned int *)(topk_lds + 64 * k);
    const int lane = threadIdx.x;
    for (int gi = blockIdx.x; gi < n_graphs; gi += gridDim.x) {
        const int sa = sfirst[gi], ns = sfirst[gi + 1] - sa;  // ns <= 64
        if (ns == 1) continue;  // (k_topk_seg wrote it)
        const int cnt = lane < ns ? c_cnt[sa + lane] : 0;
        // a key that k keys reach: lane S l + s samples list l at depth
        // (s + 1) step - 1, so each sample stands for step keys, and the
        // ceil(k / step)-th largest sample is reached by k (with k lists or
        // more, the samples are the heads)
        unsigned long long kh = 0ull;
        unsigned int kl = 0u;
        const int S = ns >= k || ns < 1 ? 1 : 64 / ns, step = ns >= k ? 1 : (k + S - 1) / S;
        const int sl = lane / S, depth = (lane % S + 1) * step - 1;
        const int scnt = __shfl(cnt, min(sl, 63));
        const bool sample = sl < ns && depth < scnt;
        const long long sat = (long long)(sa + sl) * k + depth;
        const bool bound = lane_kth(sample, sample ? c_hi[sat] : 0ull, sample ? c_lo[sat] : 0u, (k + step - 1) / step,
                                    kh, kl);
        int n = 0;
        const int total = ns * k;
        const long long base = (long long)sa * k;
        for (int i0 = 0; i0 < total; i0 += 64 * kMergePer) {  // the graph's lists lie together
            unsigned long long h[kMergePer];
            unsigned int l[kMergePer];
#pragma unroll
            for (int j = 0; j < kMergePer; ++j) {
                const long long i = base + min(i0 + 64 * j + lane, total - 1);
                h[j] = c_hi[i];
                l[j] = c_lo[i];
            }
#pragma unroll
            for (int j = 0; j < kMergePer; ++j) {
                const int i = i0 + 64 * j + lane, li = min(i / k, 63);
                const int have = __shfl(cnt, li);
                const bool c = i < total && i - li * k < have && !(bound && key_gt(kh, kl, h[j], l[j]));
                const unsigned long long m = __ballot(c);
                if (c) {
                    const int q = n + __popcll(m & ((1ull << lane) - 1ull));
                    ch[q] = h[j];
                    cl[q] = l[j];
                }
                n += __popcll(m);
            }
        }
        wave_sync();
        place_candidates(ch, cl, n, k, [&](int rank, unsigned long long h, unsigned int l) {
            ids[(long long)gi * k + rank] = (int32_t)(0xffffffffu - l);
            scores[(long long)gi * k + rank] = __longlong_as_double((long long)h);
        });
        if (lane == 0) counts[gi] = min(n, k);
        wave_sync();  // the next graph's candidates
    }
}

rs_status launch_topk_graphs(rs_graph *g, int64_t k, int32_t *d_ids, double *d_scores, int64_t *d_counts) {
    DeviceGraph &D = g->d;
    if (g->n_graphs <= 0) return RS_OK;
    hipEvent_t ev = nullptr;
    timing_begin(g, K_TOPK_GRAPHS, &ev);
    if (g->n_segs > 0) {
        hipLaunchKernelGGL(k_topk_seg, dim3((g->n_segs + kBlock / 64 - 1) / (kBlock / 64)), dim3(kBlock), 0,
                           g->stream, D.R, D.new2old, D.alive, D.vstart, D.seg_g, D.sfirst, g->n_segs, (int)k,
                           D.c_hi, D.c_lo, D.c_cnt, d_ids, d_scores, d_counts);
        if (g->n_segs > g->n_graphs_seg || g->n_graphs > g->n_graphs_seg) // several segments, or none
            hipLaunchKernelGGL(k_topk_merge, dim3(grid_for(g->n_graphs, 1, 1 << 20)), dim3(64), (size_t)(12 * 64 * k),
                           g->stream, D.c_hi, D.c_lo, D.c_cnt, D.sfirst, g->n_graphs, (int)k, d_ids, d_scores,
                           d_counts);
    } else {
        hipLaunchKernelGGL(k_topk_graphs, dim3(grid_for(g->n_graphs, 1, 1 << 20)), dim3(64), (size_t)(12 * 64 * k),
                           g->stream, D.R, D.new2old, D.alive, D.vstart, D.gorder, g->n_graphs, (int)k, d_ids,
                           d_scores, d_counts);
    }
    timing_end(g, K_TOPK_GRAPHS, ev);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "batched top-k launch");
}

// ============================================================ removals
// A removed CSR entry is marked by complementing it (~x < 0), which keeps
// every row ordered on the decoded value until the compaction below.
__device__ __forceinline__ int decode(int x) { return x < 0 ? ~x : x; }

// The out-lists that a removal must update, and the marks of the vertices
// whose rows change (bit kRowChanged).
struct OutLists {
    const int32_t *lab;
    const int64_t *oo;
    int32_t *outl;
    unsigned int *vmark;
};

// Delete the undirected edge {a, b}; the entry in the row of min(a, b) is
// the owner and decides which request wins.  Returns 1 if deleted here; nx
// and ny tell whether the rows of min(a, b) and max(a, b) were marked changed
// here first.  A deleted edge between communities also leaves the out-list
// that holds it.
template <typename OffT>
__device__ __forceinline__ int delete_edge(const OffT *off, const int32_t *deg, int32_t *col, const OutLists &O,
                                           int a, int b, bool &nx, bool &ny) {
    const int x = min(a, b), y = max(a, b);
    // y in x's row and x in y's, and the same in the out-lists of an edge
    // between communities, searched together (entries keep their places until
    // the compaction, so the positions stay valid)
    const long long xb = (long long)off[x], yb = (long long)off[y], xo = (long long)O.oo[x], yo = (long long)O.oo[y];
    const bool foreign = O.lab[x] != O.lab[y];
    const int32_t *rows[4] = {col + xb, col + yb, O.outl + xo, O.outl + yo};
    const int ds[4] = {deg[x], deg[y], foreign ? (int)(O.oo[x + 1] - xo) : 0, foreign ? (int)(O.oo[y + 1] - yo) : 0};
    const int keys[4] = {y, x, y, x};
    int k[4];
    lower_n<4, true>(rows, ds, keys, k);
    if (k[0] >= ds[0] || decode(col[xb + k[0]]) != y) return 0;
    if (atomicCAS(&col[xb + k[0]], y, ~y) != y) return 0;
    // only the request that deleted the edge gets here
    if (k[1] < ds[1] && decode(col[yb + k[1]]) == x) col[yb + k[1]] = ~x;
    nx = (atomicOr(&O.vmark[x], kRowChanged) & kRowChanged) == 0u;
    ny = (atomicOr(&O.vmark[y], kRowChanged) & kRowChanged) == 0u;
    if (k[2] < ds[2] && O.outl[xo + k[2]] == y)
        O.outl[xo + k[2]] = ~y;
    else if (k[3] < ds[3] && O.outl[yo + k[3]] == x)
        O.outl[yo + k[3]] = ~x;
    return 1;
}

// What the removals append to: the changed rows and, one by one, their chunks
// of 64 foreign entries (row's list index, chunk), at least one per row.  The
// chunks count the row's slots; those beyond its foreign list are empty.
struct ChangedRows {
    const int32_t *deg, *goff;
    int32_t *list;
    int2 *chunks;
    unsigned long long *ictr;
};

// The rows first marked changed by a wavefront's lanes, appended to the list
// of changed rows with their chunks (any order; one atomic per wavefront for
// each).  All lanes call it.
__device__ __forceinline__ void append_changed(int x, bool nx, int y, bool ny, const ChangedRows &C) {
    const int lane = (int)__lane_id();
    const unsigned long long mx = __ballot(nx), my = __ballot(ny);
    const int tot = __popcll(mx) + __popcll(my);
    if (tot == 0) return;
    const int cx = nx ? max(1, (C.goff[x + 1] - C.goff[x] + 63) >> 6) : 0;
    const int cy = ny ? max(1, (C.goff[y + 1] - C.goff[y] + 63) >> 6) : 0;
    int incl = cx + cy;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    unsigned long long first = 0, chunk = 0;
    if (lane == 63) {
        first = atomicAdd(&C.ictr[kIcChanged], (unsigned long long)tot);
        chunk = atomicAdd(&C.ictr[kIcChunks], (unsigned long long)incl);
    }
    first = __shfl(first, 63);
    chunk = __shfl(chunk, 63) + (unsigned long long)(incl - cx - cy);
    const unsigned long long below = (1ull << lane) - 1ull;
    const long long ix = (long long)first + __popcll(mx & below);
    const long long iy = (long long)first + __popcll(mx) + __popcll(my & below);
    if (nx) C.list[ix] = x;
    if (ny) C.list[iy] = y;
    for (int c = 0; c < cx; ++c) C.chunks[chunk + c] = make_int2((int)ix, c);
    for (int c = 0; c < cy; ++c) C.chunks[chunk + cx + c] = make_int2((int)iy, c);
}

// The first edge_blocks workgroups take the listed edges, a lane each; the
// others the listed vertices, a wavefront each: delete every incident edge,
// then mark the vertex dead.
template <typename OffT>
__global__ __launch_bounds__(256) void k_remove(const OffT *off, int32_t *col, OutLists O, uint8_t *alive,
                                                ChangedRows C, const int32_t *src, const int32_t *dst, long long m,
                                                int edge_blocks, const int32_t *verts, long long nv) {
    const int lane = (int)__lane_id();
    if ((int)blockIdx.x < edge_blocks) {
        unsigned long long cnt = 0;
        for (long long base = (long long)blockIdx.x * blockDim.x + threadIdx.x - lane; base < m;
             base += (long long)edge_blocks * blockDim.x) {
            const long long i = base + lane;
            int a = 0, b = 0;
            bool nx = false, ny = false;
            if (i < m) {
                a = src[i];
                b = dst[i];
                if (a != b) cnt += (unsigned long long)delete_edge(off, C.deg, col, O, a, b, nx, ny);
            }
            append_changed(min(a, b), nx, max(a, b), ny, C);
        }
        for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
        if (lane == 0 && cnt) atomicAdd(&C.ictr[kIcEdges], cnt);
        return;
    }
    const long long wave = ((long long)((int)blockIdx.x - edge_blocks) * blockDim.x + threadIdx.x) >> 6;
    const long long nwave = ((long long)((int)gridDim.x - edge_blocks) * blockDim.x) >> 6;
    for (long long i = wave; i < nv; i += nwave) {
        const int x = verts[i];
        const long long rb = (long long)off[x];
        const int d = C.deg[x];
        unsigned long long cnt = 0;
        for (int j0 = 0; j0 < d; j0 += 64) {
            const int j = j0 + lane;
            const int y = j < d ? col[rb + j] : -1;
            bool nx = false, ny = false;
            if (y >= 0) cnt += (unsigned long long)delete_edge(off, C.deg, col, O, x, y, nx, ny);
            append_changed(min(x, y), nx, max(x, y), ny, C);
        }
        for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
        if (lane == 0) {
            if (cnt) atomicAdd(&C.ictr[kIcVertexEdges], cnt);
            if (alive[x]) {
                alive[x] = 0;
                atomicAdd(&C.ictr[kIcVertices], 1ull);
            }
        }
    }
}

static OutLists out_lists(rs_graph *g) {
    OutLists O;
    O.lab = g->d.lab;
    O.oo = g->d.oo;
    O.outl = g->d.outl;
    O.vmark = g->d.vmark;
    return O;
}

rs_status launch_remove(rs_graph *g, const int32_t *src, const int32_t *dst, int64_t m, const int32_t *verts,
                        int64_t nv) {
    DeviceGraph &D = g->d;
    const int eb = m > 0 ? grid_for(m, 256, 4096) : 0, vb = nv > 0 ? grid_for(nv, 4, 4096) : 0;
    if (eb + vb == 0) return RS_OK;
    const ChangedRows C = {D.deg, D.goff, D.elist, D.echunk, D.ictr};
    if (D.off64)
        hipLaunchKernelGGL(k_remove<long long>, dim3(eb + vb), dim3(256), 0, g->stream, (const long long *)D.off,
                           D.col, out_lists(g), D.alive, C, src, dst, (long long)m, eb, verts, (long long)nv);
    else
        hipLaunchKernelGGL(k_remove<int32_t>, dim3(eb + vb), dim3(256), 0, g->stream, (const int32_t *)D.off, D.col,
                           out_lists(g), D.alive, C, src, dst, (long long)m, eb, verts, (long long)nv);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "removal launch");
}

// ------------------------------------------------------------ incremental re-score
// After a removal batch only some results change.  With E the vertices whose
// rows changed (endpoints of removed edges), a vertex u needs a new score iff
//   u is in E, or u has a foreign neighbour in E (u's pair facts, type-I
//   weights or out-lists involve it), or u is in the community of some v in
//   E and adjacent to a foreign neighbour w of v (u's pair (u, w) sums a_v);
// rows need recomputing only for E, and links only for E's entries and the
// neighbours' links back to E.  The removal kernels list E as they mark it.
// The row tiles and hub chunks that hold changed rows or affected hubs are
// rerun whole, with the block indices of the full launch, and the affected
// tile vertices are rescored in units built for the pass; every result and
// every partial is what a full pass would give.

// Compact the listed changed rows (removed entries are complemented, < 0):
// one wavefront per row, kCompactGroups groups of 64 entries loaded at once
// (a hub's long row takes one round trip per 1,024 entries), each group
// packed by a ballot and prefix (the foreign ones also into the row's slots);
// the freed tail of the capacity is set to -1.  The row's facts follow at
// once, so the marks read every foreign list's length from them.
constexpr int kCompactGroups = 16;
template <typename OffT>
__global__ __launch_bounds__(kBlock) void k_compact_rows(const OffT *off, int32_t *deg, int32_t *col, int32_t *clab,
                                                         const int32_t *lab, const int32_t *goff, int32_t *fcol,
                                                         VMeta *meta, const int32_t *list,
                                                         const unsigned long long *count) {
    const long long nl = (long long)*count;
    const int lane = threadIdx.x & 63;
    for (long long i = ((long long)blockIdx.x * kBlock + threadIdx.x) >> 6; i < nl;
         i += ((long long)gridDim.x * kBlock) >> 6) {
        const int v = list[i];
        const long long rb = (long long)off[v];
        const int d = deg[v];
        const int cv = lab[v], go = goff[v];
        int w = 0, wf = 0, p = 0;  // entries kept, foreign ones, those of them before the own run
        for (int j0 = 0; j0 < d; j0 += 64 * kCompactGroups) {  // groups of 64 entries loaded at once
            int x[kCompactGroups], c[kCompactGroups];
#pragma unroll
            for (int t = 0; t < kCompactGroups; ++t) {
                const int j = j0 + 64 * t + lane;
                x[t] = j < d ? col[rb + j] : -1;
                c[t] = j < d ? clab[rb + j] : -1;
            }
#pragma unroll
            for (int t = 0; t < kCompactGroups; ++t) {
                const unsigned long long m = __ballot(x[t] >= 0), mf = __ballot(x[t] >= 0 && c[t] != cv);
                const unsigned long long lt = (1ull << lane) - 1ull;
                p += __popcll(__ballot(x[t] >= 0 && c[t] != cv && x[t] < v));
                if (x[t] >= 0) {
                    const long long to = rb + w + __popcll(m & lt);
                    col[to] = x[t];
                    clab[to] = c[t];
                    if (c[t] != cv) fcol[go + wf + __popcll(mf & lt)] = x[t];
                }
                w += __popcll(m);
                wf += __popcll(mf);
            }
        }
        for (int j = w + lane; j < d; j += 64) {
            col[rb + j] = -1;
            clab[rb + j] = -1;
        }
        if (lane == 0) {
            deg[v] = w;
            VMeta m = meta[v];  // (ell comes with the row pass)
            m.deg = w;
            m.p = p;
            m.q = p + w - wf;
            meta[v] = m;
        }
    }
}

// Item g of a wavefront's flattened work: its owner lane (pre: the lanes'
// inclusive item counts, in LDS) and its index among the owner's items.
__device__ __forceinline__ int flat_owner(const int *pre, int g, int &idx) {
    int lo = 0, hi = 63;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (pre[mid] > g)
            hi = mid;
        else
            lo = mid + 1;
    }
    idx = g - (lo > 0 ? pre[lo - 1] : 0);
    return lo;
}

// Longest changed row whose triangles at a hub neighbour are listed pair by
// pair; a hub next to a longer changed row is rescored whole.
constexpr int kTriRow = 512;

// After removals, one wavefront per chunk of 64 entries (v, w) of a changed
// (compacted) row v's foreign list (chunks: append_changed):
// * links: v's link for the entry, and the leader and slot in v's list, which
//   moved with v's row, in w's link back to v;
// * marks: v is affected whole.  The pairs whose terms read v's row are
//   (a) (w, v) itself (w's pair facts, out-list scan, a-run),
//   (b) (w, y) for each y adjacent to both, in a third community (the
//       triangle {w, y, v} reads v's record weights),
//   (c) (x, w) for each member x of C(v) in w's row (its a-run sums a_v).
//   A tile vertex with such a pair is affected whole (its unit reruns); a
//   score hub whose own row did not change flags only the chunks holding the
//   pairs (the others keep their partials), so a changed vertex next to a
//   hub costs a few chunks, not the hub.
// Dependent loads bound it, so the searches run on the foreign lists (a tenth
// of the rows at a mixing of 0.1, which also leaves fewer chunks) and the long
// lists of (b) and (c) are worked by the whole wavefront, kMarkItems items a
// lane at once (flattened over the lanes): 205 ids removed at n = 1 million
// 21 us, 39 on whole rows one item at a time (1, 4 or 8 items, or searches of
// four ways: the same there).  Only the kRowChanged bits, set by the removals
// before, are read.
constexpr int kMarkItems = 4;
__global__ __launch_bounds__(kBlock) void k_mark_link(LinkArgs L, unsigned int *vmark, const int32_t *vscore,
                                                      const int32_t *hub_first, uint8_t *cflag, const int32_t *rows,
                                                      const int2 *chunks, const unsigned long long *n_chunks) {
    __shared__ int s_pre[kBlock / 64][64];
    const long long nc = (long long)*n_chunks;
    const int lane = threadIdx.x & 63;
    int *pre = s_pre[threadIdx.x >> 6];
    for (long long q = ((long long)blockIdx.x * kBlock + threadIdx.x) >> 6; q < nc;
         q += ((long long)gridDim.x * kBlock) >> 6) {
        const int2 it = chunks[q];
        const int v = rows[it.x];
        if (it.y == 0 && lane == 0) atomicOr(&vmark[v], kAffected);
        const VMeta mv = L.meta[v];
        const int gv = L.goff[v], fv = L.goff[v + 1] - gv;  // fv: the load-time foreign degree
        const int cv = L.lab[v], dfv = mv.deg - (mv.q - mv.p);
        const int32_t *rowv = L.fcol + gv;
        const int j = it.y * 64 + lane;
        if (it.y * 64 >= dfv) continue;
        const int id0 = L.cstart[cv], id1 = L.cstart[cv + 1];
        const bool in = j < dfv;
        int w = 0, cw = cv, gw = 0, dfw = 0, k0 = 0, k1 = 0, wh = 0;
        bool whub = false;  // w: a score hub with its row unchanged
        if (in) {
            w = rowv[j];
            cw = L.lab[w];
            gw = L.goff[w];
            const int fw = L.goff[w + 1] - gw, sw = vscore[w];
            const unsigned int mkw = L.vmark[w];
            const VMeta mw = L.meta[w];
            dfw = mw.deg - (mw.q - mw.p);
            // the out-list entry of {v, w} is in the list of the lower rank:
            // load-time foreign degree, then id
            const bool v_low = fv < fw || (fv == fw && v < w);
            const int a = v_low ? v : w, bkey = v_low ? w : v;
            const long long o0 = L.oo[a], wo = v_low ? L.oo[w] : o0;
            const int won = (int)(L.oo[w + 1] - wo), od = v_low ? (int)(L.oo[v + 1] - o0) : won;
            // in w's foreign list: C(v)'s run [k[0], k[1]) and the entry
            // (w, v) at k[2]; in v's: the start of C(w)'s run at k[3]; the
            // out-list entry at k[4]
            const int32_t *roww = L.fcol + gw;
            const int32_t *rws[5] = {roww, roww, roww, rowv, L.outl + o0};
            const int ds[5] = {dfw, dfw, dfw, dfv, od};
            const int keys[5] = {id0, id1, v, L.cstart[cw], bkey};
            int k[5];
            lower_n<5, true>(rws, ds, keys, k);
            k0 = k[0];
            k1 = k[1];
            const int kw = k[2], sv = gv + j, sw_ = gw + kw;
            const int ldv = gv + k[3], ldw = gw + k0;  // the runs' leaders
            PairLink pl;
            pl.lead = ldw;
            pl.slot = sw_;
            pl.oo = (int)wo;
            pl.on = won;
            L.plink[sv] = pl;
            L.plink[sw_].lead = ldv;
            L.plink[sw_].slot = sv;
            if (k[4] < od && L.outl[o0 + k[4]] == bkey) {
                OutEnt e;
                e.xy = v_low ? ldv : ldw;
                e.yx = v_low ? ldw : ldv;
                L.oe[o0 + k[4]] = e;
            }
            whub = sw < 0 && !(mkw & kRowChanged);
            if (whub) {
                wh = -1 - sw;
                cflag[hub_first[wh] + kw / kScoreTileP] = 1;  // (a)
            } else {
                atomicOr(&vmark[w], kAffected);
            }
        }
        // (c) the runs of C(v) in the foreign neighbours' lists: a score hub
        // whose row did not change flags the chunk holding the pair (x, w)
        // (w's place in x's foreign list); any other x is affected whole
        {
            const int cnt = k1 - k0;
            int incl = cnt;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o);
                if (lane >= o) incl += y;
            }
            pre[lane] = incl;
            const int total = __shfl(incl, 63);
            wave_sync();
            for (int g0 = 0; g0 < total; g0 += 64 * kMarkItems) {
                int x[kMarkItems], wx[kMarkItems], sx[kMarkItems];
#pragma unroll
                for (int t = 0; t < kMarkItems; ++t) {
                    const int g = g0 + 64 * t + lane;
                    int idx = 0, l = 0;
                    if (g < total) l = flat_owner(pre, g, idx);
                    const int at = __shfl(gw + k0, l);
                    wx[t] = __shfl(w, l);
                    x[t] = g < total ? L.fcol[at + idx] : -1;
                }
#pragma unroll
                for (int t = 0; t < kMarkItems; ++t) sx[t] = x[t] >= 0 ? vscore[x[t]] : 0;
#pragma unroll
                for (int t = 0; t < kMarkItems; ++t) {
                    if (x[t] < 0) continue;
                    if (sx[t] < 0 && !(L.vmark[x[t]] & kRowChanged)) {
                        const VMeta m = L.meta[x[t]];
                        const int32_t *row[1] = {L.fcol + L.goff[x[t]]};
                        const int d[1] = {m.deg - (m.q - m.p)};
                        const int key[1] = {wx[t]};
                        int kx[1];
                        lower_n<1, false>(row, d, key, kx);
                        cflag[hub_first[-1 - sx[t]] + kx[0] / kScoreTileP] = 1;
                    } else {
                        atomicOr(&vmark[x[t]], kAffected);
                    }
                }
            }
            wave_sync();
        }
        // (b) the triangles {w, y, v} at the hub neighbours w: the pairs
        // (w, y) for the foreign neighbours y of v in a third community
        const unsigned long long hubs = __ballot(whub);
        if (hubs) {
            if (mv.deg > kTriRow) {  // too long to intersect: the hub reruns whole
                if (whub) atomicOr(&vmark[w], kAffected);
            } else {
                const int cnt = whub ? dfv : 0;
                int incl = cnt;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int y = __shfl_up(incl, o);
                    if (lane >= o) incl += y;
                }
                pre[lane] = incl;
                const int total = __shfl(incl, 63);
                wave_sync();
                for (int g0 = 0; g0 < total; g0 += 64 * kMarkItems) {
                    const int32_t *row[kMarkItems];
                    int d[kMarkItems], key[kMarkItems], hl[kMarkItems], k[kMarkItems], cwl[kMarkItems];
#pragma unroll
                    for (int t = 0; t < kMarkItems; ++t) {
                        const int g = g0 + 64 * t + lane;
                        int idx = 0, l = 0;
                        if (g < total) l = flat_owner(pre, g, idx);
                        cwl[t] = __shfl(cw, l);
                        hl[t] = __shfl(wh, l);
                        row[t] = L.fcol + __shfl(gw, l);
                        d[t] = __shfl(dfw, l);
                        key[t] = g < total ? rowv[idx] : -1;
                    }
#pragma unroll
                    for (int t = 0; t < kMarkItems; ++t)
                        if (key[t] < 0 || L.lab[key[t]] == cwl[t]) d[t] = 0;
                    lower_n<kMarkItems, false>(row, d, key, k);
#pragma unroll
                    for (int t = 0; t < kMarkItems; ++t)
                        if (k[t] < d[t] && row[t][k[t]] == key[t]) cflag[hub_first[hl[t]] + k[t] / kScoreTileP] = 1;
                }
                wave_sync();
            }
        }
    }
}

// Marks -> units: a changed row flags its row block; an affected hub flags
// all chunks of its score hub; an affected tile vertex is placed in abin,
// grouped by the bin of its load-time foreign degree (units of rescored
// vertices are built per pass, so scattered affected vertices do not rerun
// whole tiles).  Two launches over contiguous vertex ranges, one range per
// workgroup, so that no counter in global memory is shared: count per range
// and bin (LDS atomics), then each range sums the counts before its own
// (18 KB a workgroup, from the L2; a launch of its own for the sums took 8 us
// and a gap) and places its vertices there.  Placement clears the marks, and
// beside it other workgroups turn the flags into lists.
__device__ __forceinline__ int score_bin(long long fgn) {
    int b = 0;
    while (b < kScoreBins - 1 && (1ll << b) < fgn) ++b;
    return b;
}

__device__ __forceinline__ void unit_range(long long n, int groups, long long &lo, long long &hi) {
    const long long per = ((n + groups - 1) / groups + 63) & ~63ll;
    lo = min(n, (long long)blockIdx.x * per);
    hi = min(n, lo + per);
}

// The marks of kMarkPer vertices of a range per thread, loaded together (a
// loop that tests each mark before loading the next waits for every load):
// slots past the range load its last mark and are skipped by the caller.
constexpr int kMarkPer = 8;
__device__ __forceinline__ void load_marks(const unsigned int *vmark, long long v0, long long hi,
                                           unsigned int (&mk)[kMarkPer]) {
#pragma unroll
    for (int j = 0; j < kMarkPer; ++j) {
        const long long v = v0 + (long long)j * kBlock;
        mk[j] = vmark[v < hi ? v : hi - 1];
    }
}

// ucnt[r * kUnitGroups + range]: rows 0..kScoreBins-1 tile vertices per bin,
// row kScoreBins affected vertices.
__global__ __launch_bounds__(kBlock) void k_units_count(const unsigned int *vmark, const int32_t *vrowb,
                                                        const int32_t *vscore, const int32_t *goff, long long n,
                                                        uint8_t *rflag, uint8_t *hflag, int32_t *ucnt) {
    __shared__ int s_cnt[kUnitRows];
    if (threadIdx.x < kUnitRows) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    long long lo, hi;
    unit_range(n, (int)gridDim.x, lo, hi);
    int aff = 0;
    for (long long v0 = lo + threadIdx.x; v0 < hi; v0 += (long long)kMarkPer * kBlock) {
        unsigned int mk[kMarkPer];
        load_marks(vmark, v0, hi, mk);
#pragma unroll
        for (int j = 0; j < kMarkPer; ++j) {
            const long long v = v0 + (long long)j * kBlock;
            const unsigned int m = mk[j];
            if (v >= hi || !m) continue;
            if (m & kRowChanged) rflag[vrowb[v]] = 1;
            if (m & kAffected) {
                ++aff;
                const int sc = vscore[v];
                if (sc >= 0)
                    atomicAdd(&s_cnt[score_bin(goff[v + 1] - goff[v])], 1);
                else
                    hflag[-1 - sc] = 1;
            }
        }
    }
    if (aff) atomicAdd(&s_cnt[kScoreBins], aff);
    __syncthreads();
    if (threadIdx.x < kUnitRows) ucnt[threadIdx.x * kUnitGroups + blockIdx.x] = s_cnt[threadIdx.x];
}

// Append the lanes' values whose pred holds to list (one atomic per
// wavefront; all lanes call it).
__device__ __forceinline__ void wave_append(bool pred, int val, int32_t *list, unsigned long long *count) {
    const int lane = threadIdx.x & 63;
    const unsigned long long m = __ballot(pred);
    if (!m) return;
    unsigned long long first = 0;
    if (lane == 0) first = atomicAdd(count, (unsigned long long)__popcll(m));
    first = __shfl(first, 0);
    if (pred) list[first + __popcll(m & ((1ull << lane) - 1ull))] = val;
}

// The flags' part of k_units_place.
struct UnitLists {
    uint8_t *rflag, *cflag;
    const uint8_t *hflag;
    const int2 *hub_chunk;
    int n_rows, n_chunks, n_chunks_lds;
    int32_t *rlist, *slist, *hlist;
};

// Flags -> the incremental launches' lists (indices of the full launches):
// the flagged row blocks, and the score-hub chunks to rerun, each chunk of a
// hub flagged whole and each chunk flagged by itself (the main list takes
// the LDS-hub chunks, the big list the others).  Clears the row and chunk
// flags; the hub flags are cleared by the score pass that follows.
__device__ __forceinline__ void unit_lists(const UnitLists &U, int block, int blocks, unsigned long long *ictr) {
    const int lane = threadIdx.x & 63;
    const int top = max(U.n_rows, U.n_chunks);
    for (int base = block * kBlock + (threadIdx.x & ~63); base < top; base += blocks * kBlock) {
        const int i = base + lane;
        const bool r = i < U.n_rows && U.rflag[i] != 0;
        if (r) U.rflag[i] = 0;
        bool c = false;
        if (i < U.n_chunks) {
            const bool own = U.cflag[i] != 0;
            if (own) U.cflag[i] = 0;
            c = own || U.hflag[U.hub_chunk[i].x] != 0;
        }
        wave_append(r, i, U.rlist, &ictr[kIcRows]);
        wave_append(c && i < U.n_chunks_lds, i, U.slist, &ictr[kIcMain]);
        wave_append(c && i >= U.n_chunks_lds, i - U.n_chunks_lds, U.hlist, &ictr[kIcBig]);
    }
}

// The first `groups` workgroups place their range's affected tile vertices in
// their bins (any order inside a range and bin; a vertex's score does not
// depend on its unit) and clear the marks; the others make the lists.  The
// first workgroup also leaves the bins' totals and w_max before the pass in
// the counters, what the host reports in pinned memory, and the next
// re-score's counters cleared.
static_assert(kUnitGroups == 2 * kBlock, "k_units_place sums two ranges per thread");
__global__ __launch_bounds__(kBlock) void k_units_place(unsigned int *vmark, const int32_t *vscore,
                                                        const int32_t *goff, long long n, const int32_t *ucnt,
                                                        int groups, int32_t *abin, UnitLists U,
                                                        unsigned long long *ictr, unsigned long long *ictr_next,
                                                        const DevCounters *ctr, RemovalCounts *host) {
    if ((int)blockIdx.x >= groups) {
        unit_lists(U, (int)blockIdx.x - groups, (int)gridDim.x - groups, ictr);
        return;
    }
    __shared__ int s_cur[kScoreBins];
    __shared__ int s_sum[kUnitRows][2][kBlock / 64];  // before this range; of all ranges
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    {
        int2 x[kUnitRows];
        const int j = 2 * (int)threadIdx.x;
#pragma unroll
        for (int r = 0; r < kUnitRows; ++r) {
            x[r] = *(const int2 *)&ucnt[r * kUnitGroups + j];
            if (j >= groups) x[r].x = 0;
            if (j + 1 >= groups) x[r].y = 0;
        }
#pragma unroll
        for (int r = 0; r < kUnitRows; ++r) {
            int all = x[r].x + x[r].y;
            int before = (j < (int)blockIdx.x ? x[r].x : 0) + (j + 1 < (int)blockIdx.x ? x[r].y : 0);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                all += __shfl_xor(all, o);
                before += __shfl_xor(before, o);
            }
            if (lane == 0) {
                s_sum[r][0][wave] = before;
                s_sum[r][1][wave] = all;
            }
        }
    }
    __syncthreads();
    if (threadIdx.x < kUnitRows) {
        const int r = threadIdx.x;
        int at = 0, total = 0;
        for (int q = 0; q <= r; ++q) {
            at += total;
            total = 0;
            for (int w = 0; w < kBlock / 64; ++w) total += s_sum[q][1][w];
        }
        for (int w = 0; w < kBlock / 64; ++w) at += s_sum[r][0][w];
        if (r < kScoreBins) s_cur[r] = at;
        if (blockIdx.x == 0 && r < kScoreBins) ictr[kIcBins + r] = (unsigned long long)total;
        if (blockIdx.x == 0 && r == kScoreBins) {
            ictr[kIcWmaxOld] = ctr->wmax_bits;
            host->edges = ictr[kIcEdges];
            host->vertex_edges = ictr[kIcVertexEdges];
            host->vertices = ictr[kIcVertices];
            host->affected = (unsigned long long)total;
            __threadfence_system();
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < kIcCount) ictr_next[threadIdx.x] = 0ull;
    __syncthreads();
    long long lo, hi;
    unit_range(n, groups, lo, hi);
    for (long long v0 = lo + threadIdx.x; v0 < hi; v0 += (long long)kMarkPer * kBlock) {
        unsigned int mk[kMarkPer];
        load_marks(vmark, v0, hi, mk);
#pragma unroll
        for (int j = 0; j < kMarkPer; ++j) {
            const long long v = v0 + (long long)j * kBlock;
            const unsigned int m = mk[j];
            if (v >= hi || !m) continue;
            vmark[v] = 0u;
            if ((m & kAffected) && vscore[v] >= 0)
                abin[atomicAdd(&s_cur[score_bin(goff[v + 1] - goff[v])], 1)] = (int32_t)v;
        }
    }
}

template <typename OffT>
static rs_status incremental_marks_t(rs_graph *g) {
    DeviceGraph &D = g->d;
    if (D.n == 0) return RS_OK;
    const OffT *off = (const OffT *)D.off;
    const int gn = grid_for(D.n, kBlock, 1024);
    hipLaunchKernelGGL(k_compact_rows<OffT>, dim3(gn), dim3(kBlock), 0, g->stream, off, D.deg, D.col, D.clab,
                       D.lab, D.goff, D.fcol, D.meta, D.elist, &D.ictr[kIcChanged]);
    hipLaunchKernelGGL(k_mark_link, dim3(gn), dim3(kBlock), 0, g->stream, link_args(g), D.vmark,
                       (const int32_t *)D.vscore, (const int32_t *)D.shub_first, D.cflag, D.elist, D.echunk,
                       &D.ictr[kIcChunks]);
    const int ug = grid_for(D.n, kBlock, kUnitGroups);
    hipLaunchKernelGGL(k_units_count, dim3(ug), dim3(kBlock), 0, g->stream, D.vmark, D.vrowb, D.vscore, D.goff,
                       (long long)D.n, D.rflag, D.hflag, D.ucnt);
    UnitLists U;
    U.rflag = D.rflag;
    U.cflag = D.cflag;
    U.hflag = D.hflag;
    U.hub_chunk = D.shub_chunk;
    U.n_rows = g->grid_rows;
    U.n_chunks = g->n_schunks;
    U.n_chunks_lds = g->n_schunks_lds;
    U.rlist = D.rlist;
    U.slist = D.slist;
    U.hlist = D.hlist;
    const int lg = grid_for(std::max(g->grid_rows, g->n_schunks), kBlock, 4096);
    hipLaunchKernelGGL(k_units_place, dim3(ug + lg), dim3(kBlock), 0, g->stream, D.vmark, D.vscore, D.goff,
                       (long long)D.n, D.ucnt, ug, D.abin, U, D.ictr, D.ictr_next, D.ctr, g->rem_cnt_host);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "incremental marks launch");
}

rs_status launch_incremental_marks(rs_graph *g) {
    return g->d.off64 ? incremental_marks_t<long long>(g) : incremental_marks_t<int32_t>(g);
}

// ============================================================ readers
__global__ void k_gather_scores(const double *R, const int32_t *new2old, const DevCounters *ctr,
                                const unsigned long long *gwmax, const int32_t *vgraph, long long n, int raw,
                                double *out) {
    const double wmax = bitsd(ctr->wmax_bits);
    for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (long long)gridDim.x * blockDim.x)
        out[new2old[v]] = raw ? R[v] * (gwmax ? bitsd(gwmax[vgraph[v]]) : wmax) : R[v];
}

rs_status launch_gather_scores(rs_graph *g, double *d_out, int raw) {
    const int grid = grid_for(g->d.n, 256, 8192);
    hipLaunchKernelGGL(k_gather_scores, dim3(grid), dim3(256), 0, g->stream, g->d.R, g->d.new2old, g->d.ctr,
                       g->n_graphs > 0 ? g->d.gwmax : nullptr, g->d.vgraph, (long long)g->d.n, raw, d_out);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "gather launch");
}

// The per-vertex results in caller order (any array may be null).  A vertex
// without foreign neighbours counts no triads.
__global__ __launch_bounds__(kBlock) void k_gather_counts(const VMeta *meta, const long long *tI, const long long *tII,
                                                          const double *wown, const int32_t *new2old, long long n,
                                                          VertexOut out) {
    for (long long v = (long long)blockIdx.x * kBlock + threadIdx.x; v < n; v += (long long)gridDim.x * kBlock) {
        const VMeta m = meta[v];
        const int x = new2old[v], dp = m.deg - (m.q - m.p);
        if (out.border) out.border[x] = dp > 0 ? 1 : 0;
        if (out.ell) out.ell[x] = m.ell;
        if (out.dprime) out.dprime[x] = dp;
        if (out.tI) out.tI[x] = dp > 0 ? tI[v] : 0;
        if (out.tII) out.tII[x] = dp > 0 ? tII[v] : 0;
        if (out.w_own) out.w_own[x] = wown[v];
    }
}

rs_status launch_gather_counts(rs_graph *g, const VertexOut &out) {
    DeviceGraph &D = g->d;
    hipLaunchKernelGGL(k_gather_counts, dim3(grid_for(D.n, kBlock, 8192)), dim3(kBlock), 0, g->stream, D.meta, D.tI,
                       D.tII, D.wown, D.new2old, (long long)D.n, out);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "gather launch");
}

rs_status launch_zero_u64(rs_graph *g, unsigned long long *p, int count) {
    hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, g->stream, p, count);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "zero launch");
}

// ============================================================ reachable communities
// For the absolute AWCC of the robustness experiments (Section VII-B): the
// connected components of the current graph, then, for each source, the
// communities of the other members of its component.
//
// Components are a union-find over the live edges, with no rounds to
// convergence and no host check: parents only ever decrease (comp[v] <= v, so no
// cycle can form), an edge hooks the larger of its two roots under the smaller
// with a compare-and-swap, and a failed one goes on from the value it met, a
// smaller id.  (Rounds of hooking and pointer jumping, with a thread walking
// each row, took four sweeps of 37 to 740 us at n = 10^5 and a host wait per
// four rounds.)  Parents may be read from a cache that another XCD's swap has
// made stale, and path stores may land late: a value once above v stays an
// ancestor of v, only roots are swapped, and no store makes a root, so a stale
// value costs a failed swap and nothing else.
__device__ __forceinline__ int32_t cc_load(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void cc_store(int32_t *p, int32_t x) {
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The root above v; every second vertex of the path is pointed at its
// grandparent on the way.
__device__ __forceinline__ int32_t cc_find(int32_t *comp, int32_t v) {
    int32_t prev = v, p = cc_load(&comp[v]);
    if (p == v) return v;
    for (;;) {
        const int32_t next = cc_load(&comp[p]);
        if (next == p) return p;
        cc_store(&comp[prev], next);
        prev = p;
        p = next;
    }
}

__device__ __forceinline__ void cc_unite(int32_t *comp, int32_t u, int32_t v) {
    int32_t a = cc_find(comp, u), b = cc_find(comp, v);
    while (a != b) {
        if (a < b) {
            const int32_t t = a;
            a = b;
            b = t;
        }
        const int32_t old = atomicCAS(&comp[a], a, b);  // a is the larger root
        if (old == a) return;
        a = cc_find(comp, old);  // a was hooked meanwhile: old < a
    }
}

// Every vertex starts under its smallest neighbour, if that is smaller.  Also
// clears the community bitmaps (n_bits words).
template <typename OffT>
__global__ __launch_bounds__(kBlock) void k_cc_init(const OffT *off, const int32_t *deg, const int32_t *col,
                                                    int32_t *comp, long long n, unsigned int *bits,
                                                    long long n_bits) {
    for (long long w = (long long)blockIdx.x * kBlock + threadIdx.x; w < n_bits; w += (long long)gridDim.x * kBlock)
        bits[w] = 0u;
    for (long long v = (long long)blockIdx.x * kBlock + threadIdx.x; v < n; v += (long long)gridDim.x * kBlock) {
        const int32_t x = deg[v] > 0 ? col[off[v]] : (int32_t)v;
        comp[v] = x >= 0 && x < (int32_t)v ? x : (int32_t)v;  // (rows are compacted after removals: x < 0 is defensive)
    }
}

// One sweep over the edges, each from its larger end (a row's entries below the
// vertex).  A wavefront takes the rows of 64 vertices, flattened over its
// lanes.  kUnite: the ends are united.  Else, with comp[] flat (roots), the
// larger root takes the smaller as its parent if that is less than what it
// has: a round of this joins most trees with two reads an edge, and after
// kCcRounds of them (each flattened) the uniting sweep meets the same root
// twice at nearly every edge.  Uniting from the start, where trees grow deep
// while every lane climbs them, took 200 to 350 us at n = 10^5 with 4.6 edges
// left a vertex (whole queries: one round 97 us, two 108, three 118).  With five
// live entries a vertex and more one round is the fastest or near it up to n =
// 400,000 (n = 400,000, mean degree 12: 245, 289 and 328 us); sparser remainders
// of large graphs would gain from more (n = 400,000 with 1.5: 1,741, 337 and 192;
// n = 1 million with 5: 1,043, 403 and 446, with 2: 3,976, 890 and 294).
constexpr int kCcRounds = 1;
template <bool kUnite, typename OffT>
__global__ __launch_bounds__(kBlock) void k_cc_hook(const OffT *off, const int32_t *deg, const int32_t *col,
                                                    int32_t *comp, long long n) {
    __shared__ int s_pre[kBlock / 64][64];
    __shared__ long long s_rb[kBlock / 64][64];
    const int lane = threadIdx.x & 63;
    int *pre = s_pre[threadIdx.x >> 6];
    long long *row = s_rb[threadIdx.x >> 6];
    auto join = [&](int32_t x, int32_t v) {
        if (x < 0 || x >= v) return;
        if (kUnite) {
            cc_unite(comp, x, v);
        } else {
            int32_t a = cc_load(&comp[x]), b = cc_load(&comp[v]);
            if (a == b) return;
            if (a < b) {
                const int32_t t = a;
                a = b;
                b = t;
            }
            if (b < cc_load(&comp[a])) atomicMin(&comp[a], b);
        }
    };
    for (long long v0 = (long long)blockIdx.x * kBlock + (threadIdx.x & ~63); v0 < n;
         v0 += (long long)gridDim.x * kBlock) {
        const long long v = v0 + lane;
        int cnt = 0;
        long long rb = 0;
        if (v < n) {
            rb = (long long)off[v];
            cnt = deg[v];
        }
        long long incl = cnt;  // (the 64 rows may hold 2^31 entries and more)
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const long long y = __shfl_up(incl, o);
            if (lane >= o) incl += y;
        }
        const long long total = __shfl(incl, 63);
        if (flat_rows_fit(total)) {
            pre[lane] = (int)incl;
            row[lane] = rb;
            wave_sync();
            for (int g0 = 0; g0 < (int)total; g0 += 64) {
                const int g = g0 + lane;
                if (g < (int)total) {
                    int j;
                    const int l = flat_owner(pre, g, j);
                    join(col[row[l] + j], (int32_t)(v0 + l));
                }
            }
            wave_sync();
        } else {
            for (int j = 0; j < cnt; ++j) join(col[rb + j], (int32_t)v);
        }
    }
}

// Point every vertex at its root.
__global__ __launch_bounds__(kBlock) void k_cc_flatten(int32_t *comp, long long n) {
    for (long long v = (long long)blockIdx.x * kBlock + threadIdx.x; v < n; v += (long long)gridDim.x * kBlock) {
        int32_t c = cc_load(&comp[v]);
        for (;;) {
            const int32_t p = cc_load(&comp[c]);
            if (p == c) break;
            c = p;
        }
        cc_store(&comp[v], c);
    }
}

// What is kept of a source until its count is known: the first source of the
// same component, whose bitmap serves the whole component, and whether
// another member shares the source's community.
struct ReachSource {
    int32_t group;
    unsigned int other;
};
static_assert(sizeof(ReachSource) == sizeof(long long), "the counts replace the sources' facts");

// One workgroup: the root of each source's component is marked with the first
// of its sources to get there (comp[root] = ~i), and the sources get their
// groups.
__global__ __launch_bounds__(kMaxReachSources) void k_reach_groups(int32_t *comp, const int32_t *src, int ns,
                                                                   ReachSource *out) {
    const int i = threadIdx.x;
    if (i < ns) {
        const int32_t c = cc_load(&comp[src[i]]);
        if (c >= 0) atomicCAS(&comp[c], c, ~i);
    }
    __syncthreads();
    if (i < ns) {  // (the swaps act in memory: read past the caches)
        const int32_t c = __hip_atomic_load(&comp[src[i]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int32_t g = c < 0 ? c : __hip_atomic_load(&comp[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        out[i].group = ~g;
        out[i].other = 0u;
    }
}

// Each member of a marked component sets its community's bit in the
// component's bitmap (in LDS when all bitmaps fit, added to the global ones at
// the end; most members find their bit set already), and tells the sources of
// the same component and community that they are not alone.
constexpr int kReachWords = 8192;
__global__ __launch_bounds__(kBlock) void k_reach_bits(const int32_t *comp, const int32_t *lab, long long n,
                                                       const int32_t *src, int ns, int words, ReachSource *rs,
                                                       unsigned int *bits) {
    __shared__ int32_t s_g[kMaxReachSources], s_v[kMaxReachSources], s_l[kMaxReachSources];
    __shared__ unsigned int s_other[kMaxReachSources], s_bits[kReachWords];
    const bool local = (long long)ns * words <= kReachWords;
    for (int i = threadIdx.x; i < ns; i += kBlock) {
        s_g[i] = rs[i].group;
        s_v[i] = src[i];
        s_l[i] = lab[src[i]];
        s_other[i] = 0u;
    }
    if (local)
        for (int i = threadIdx.x; i < ns * words; i += kBlock) s_bits[i] = 0u;
    __syncthreads();
    for (long long v = (long long)blockIdx.x * kBlock + threadIdx.x; v < n; v += (long long)gridDim.x * kBlock) {
        int32_t g = comp[v];
        const int32_t l = lab[v];
        if (g >= 0) g = comp[g];
        if (g >= 0) continue;  // no source in this component
        g = ~g;
        const unsigned int bit = 1u << (l & 31);
        const long long at = (long long)g * words + (l >> 5);
        if (local) {
            if (!(s_bits[at] & bit)) atomicOr(&s_bits[at], bit);
        } else if (!(__hip_atomic_load(&bits[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit)) {
            atomicOr(&bits[at], bit);
        }
        for (int i = 0; i < ns; ++i)
            if (s_g[i] == g && s_l[i] == l && s_v[i] != (int32_t)v) s_other[i] = 1u;
    }
    __syncthreads();
    if (local)
        for (int i = threadIdx.x; i < ns * words; i += kBlock)
            if (s_bits[i]) atomicOr(&bits[i], s_bits[i]);
    for (int i = threadIdx.x; i < ns; i += kBlock)
        if (s_other[i]) atomicOr(&rs[i].other, 1u);
}

// counts[i] (in the place of rs[i]) = the bits of source i's component, less
// its own community's when no other member has it (one wavefront per source).
__global__ __launch_bounds__(kBlock) void k_reach_counts(const unsigned int *bits, int ns, int words,
                                                         ReachSource *rs) {
    const int i = (int)blockIdx.x * (kBlock / 64) + (int)(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (i >= ns) return;
    const ReachSource s = rs[i];
    int c = 0;
    for (int w = lane; w < words; w += 64) c += __popc(bits[(long long)s.group * words + w]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if (lane == 0) ((long long *)rs)[i] = (long long)c - (s.other ? 0 : 1);
}

template <typename OffT>
static void components_t(rs_graph *g, int32_t *comp, unsigned int *bits, long long n_bits) {
    DeviceGraph &D = g->d;
    const int grid = grid_for(D.n, kBlock, 8192);
    hipLaunchKernelGGL(k_cc_init<OffT>, dim3(grid), dim3(kBlock), 0, g->stream, (const OffT *)D.off, D.deg, D.col,
                       comp, (long long)D.n, bits, n_bits);
    hipLaunchKernelGGL(k_cc_flatten, dim3(grid), dim3(kBlock), 0, g->stream, comp, (long long)D.n);
    for (int i = 0; i <= kCcRounds; ++i) {
        if (i < kCcRounds)
            hipLaunchKernelGGL((k_cc_hook<false, OffT>), dim3(grid), dim3(kBlock), 0, g->stream, (const OffT *)D.off,
                               D.deg, D.col, comp, (long long)D.n);
        else
            hipLaunchKernelGGL((k_cc_hook<true, OffT>), dim3(grid), dim3(kBlock), 0, g->stream, (const OffT *)D.off,
                               D.deg, D.col, comp, (long long)D.n);
        hipLaunchKernelGGL(k_cc_flatten, dim3(grid), dim3(kBlock), 0, g->stream, comp, (long long)D.n);
    }
}

rs_status launch_reach(rs_graph *g, const int32_t *d_src, int ns, int32_t *comp, unsigned int *bits, int words,
                       long long *d_counts) {
    DeviceGraph &D = g->d;
    if (D.off64)
        components_t<long long>(g, comp, bits, (long long)ns * words);
    else
        components_t<int32_t>(g, comp, bits, (long long)ns * words);
    ReachSource *rs = (ReachSource *)d_counts;
    hipLaunchKernelGGL(k_reach_groups, dim3(1), dim3(kMaxReachSources), 0, g->stream, comp, d_src, ns, rs);
    hipLaunchKernelGGL(k_reach_bits, dim3(grid_for(D.n, 2 * kBlock, 1024)), dim3(kBlock), 0, g->stream, comp, D.lab,
                       (long long)D.n, d_src, ns, words, rs, bits);
    hipLaunchKernelGGL(k_reach_counts, dim3((ns + kBlock / 64 - 1) / (kBlock / 64)), dim3(kBlock), 0, g->stream,
                       bits, ns, words, rs);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "reach launch");
}

// ------------------------------------------------------------ static scratch
// Device memory of rs_reachable_communities_static, the entry point for
// callers that cannot allocate: one array per device (it lives as long as
// the process), shared by every call on that device.  Host code never passes
// the array's name to a kernel -- that is a host-side stand-in, not a device
// address -- but the per-device address taken once with
// hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxDevices] = {};

rs_status static_scratch(int device, void **out) {
    *out = nullptr;
    if (device < 0 || device >= kMaxDevices) return fail(RS_ERR_ARG, "device index out of range");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e == hipSuccess && cur != device) e = hipSetDevice(device);
        void *p = nullptr;
        if (e == hipSuccess) e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur >= 0 && cur != device) (void)hipSetDevice(cur);
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        g_scratch_ptr[device] = p;
    }
    *out = g_scratch_ptr[device];
    return RS_OK;
}

}  // namespace rs
