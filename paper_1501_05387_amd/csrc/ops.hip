// ops.hip -- the frontier operators on their own, for callers that compose
// their own traversals (Sec. 3-4: advance and filter are the two operators
// every primitive is built from).
//
//   advance  a vertex frontier (any order, duplicates allowed) becomes its
//            edge frontier: for every entry u, in frontier order, every edge
//            e of u in CSR order, as (u, e, C[e]).  The entries' degrees are
//            scanned into output offsets (the scan of Sec. 4.4), the entries
//            with edges become a chunked frontier queue, and the
//            load-balanced advance writes each edge at its offset, so the
//            output order is exactly the sequential one.  An edge frontier
//            (Sec. 4.1 lets advance start from edges as well) is first
//            gathered to the edges' far ends; each output then carries the
//            input edge in place of u.
//   filter   a list of vertices (duplicates allowed) becomes the ascending
//            list of the distinct vertices not excluded by a byte mask:
//            items leave a mark byte (idempotent stores, Sec. 4.5), and a
//            scan over the marks compacts them in vertex order.
//   scan     the exact exclusive prefix sum (uint64) of a uint32 array: the
//            scan that turns degrees into output offsets (Sec. 4.4), alone.
//   split    the near/far split of a frontier (Sec. 4.5, priority queue):
//            items whose distance is below a threshold go to the near list,
//            the others to the far list, both in input order (one scan of
//            the pair (near, far) gives every item its slot).
//
// The scans run in two launches: per-tile totals, and a pass in which every
// work-group adds up the tiles before its own, recomputes its tile's prefix and
// writes.  Each thread owns SCAN_EPT consecutive elements, so every write lands
// at its exclusive prefix.  Past SELF_TILES tiles, where reading all totals in
// every work-group would cost more than a launch, one work-group scans them in
// between.
//
// A call on an ordinary frontier is launches and waits, not bytes, so it waits
// for the device once: ids out of range are noted by the pass that first reads
// them (and give nothing there), and the writing passes compare the grand total
// with the capacity on the device and write nothing when it is exceeded or an
// id was bad.  On R-MAT with 260,017 vertices, an advance of 3,781
// vertices (180 K edges), a filter of the result and a split of what is left
// took 74, 65 and 66 us with a wait for each of these checks, 57, 46 and 46 us
// so (43, 33 and 33 with the wait of read_back since).
#include <string.h>

#include <algorithm>
#include <string>

#include "compact.h"
#include "engine.h"

namespace gfr {

constexpr int SCAN_EPT = 8;
constexpr int64_t SCAN_TILE = (int64_t)GFR_BLOCK * SCAN_EPT;
constexpr int64_t SELF_TILES = 1024;   // 2 M elements

struct P2 {
    unsigned long long a, b;   // advance: edges, queue entries; filter: unused, list entries
};

// What one read-back brings: the grand totals, and whether an id was out of range.
struct Grand {
    P2 tot;
    unsigned long long bad;
};
constexpr unsigned long long ANY = ~0ull;
constexpr unsigned long long BAD_TILE = 1ull << 63;   // in a tile total's b: the tile holds a bad id

// Whether the writing passes write: every id good, totals within the capacity.
struct Gate {
    unsigned long long cap_a, cap_b;
    __device__ bool open(const Grand &g) const { return g.bad == 0ull && g.tot.a <= cap_a && g.tot.b <= cap_b; }
};

__device__ __forceinline__ P2 block_excl_scan_p2(P2 x, P2 *total)
{
    unsigned long long ta, tb;
    P2 r;
    r.a = block_excl_scan_u64(x.a, &ta);
    r.b = block_excl_scan_u64(x.b, &tb);
    total->a = ta;
    total->b = tb;
    return r;
}

// per-tile totals
template <class Val>
__global__ __launch_bounds__(GFR_BLOCK) void scan_reduce(Val val, int64_t count, P2 *totals)
{
    const int64_t t0 = (int64_t)blockIdx.x * SCAN_TILE;
    P2 s{0, 0};
    bool wrong = false;
    for (int64_t i = t0 + threadIdx.x; i < count && i < t0 + SCAN_TILE; i += GFR_BLOCK) {
        wrong |= val.bad(i);
        const P2 x = val(i);
        s.a += x.a;
        s.b += x.b;
    }
    P2 tot;
    (void)block_excl_scan_p2(s, &tot);
    const int any = __syncthreads_or(wrong);
    if (threadIdx.x == 0) totals[blockIdx.x] = P2{tot.a, tot.b | (any ? BAD_TILE : 0ull)};
}

// exclusive scan of the tile totals in place (one work-group)
__global__ __launch_bounds__(GFR_BLOCK) void scan_totals(P2 *totals, int64_t ntiles, Grand *grand)
{
    P2 carry{0, 0};
    bool wrong = false;
    for (int64_t b0 = 0; b0 < ntiles; b0 += GFR_BLOCK) {
        const int64_t i = b0 + threadIdx.x;
        P2 x = i < ntiles ? totals[i] : P2{0, 0};
        wrong |= x.b >= BAD_TILE;
        x.b &= ~BAD_TILE;
        P2 tot;
        const P2 ex = block_excl_scan_p2(x, &tot);
        if (i < ntiles) totals[i] = P2{carry.a + ex.a, carry.b + ex.b};
        carry.a += tot.a;
        carry.b += tot.b;
        __syncthreads();
    }
    const int any = __syncthreads_or(wrong);
    if (threadIdx.x == 0) *grand = Grand{carry, any ? 1ull : 0ull};
}

// The same from the plain totals, by every work-group for itself: the grand
// total, and in *below the sum of the tiles before this one.
__device__ __forceinline__ Grand sum_tiles(const P2 *totals, int64_t ntiles, P2 *below)
{
    P2 all{0, 0}, lo{0, 0};
    bool wrong = false;
    for (int64_t i = threadIdx.x; i < ntiles; i += GFR_BLOCK) {
        P2 x = totals[i];
        wrong |= x.b >= BAD_TILE;
        x.b &= ~BAD_TILE;
        all.a += x.a;
        all.b += x.b;
        if (i < (int64_t)blockIdx.x) {
            lo.a += x.a;
            lo.b += x.b;
        }
    }
    Grand g;
    (void)block_excl_scan_p2(all, &g.tot);
    (void)block_excl_scan_p2(lo, below);
    g.bad = __syncthreads_or(wrong) ? 1ull : 0ull;
    return g;
}

// each element with its exclusive prefix; `self`: the totals are plain, and the
// first work-group leaves the grand total
template <class Val, class Emit>
__global__ __launch_bounds__(GFR_BLOCK) void scan_emit(Val val, int64_t count, const P2 *totals, int64_t ntiles,
                                                       bool self, Grand *grand, Gate gate, Emit emit)
{
    P2 below;
    if (self) {
        const Grand g = sum_tiles(totals, ntiles, &below);
        if (blockIdx.x == 0 && threadIdx.x == 0) *grand = g;
        if (!gate.open(g)) return;
    } else {
        if (!gate.open(*grand)) return;
        below = totals[blockIdx.x];
    }
    const int64_t i0 = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_EPT;
    P2 x[SCAN_EPT];
    P2 s{0, 0};
#pragma unroll
    for (int j = 0; j < SCAN_EPT; ++j) {
        x[j] = i0 + j < count ? val(i0 + j) : P2{0, 0};
        s.a += x[j].a;
        s.b += x[j].b;
    }
    P2 tot;
    const P2 ex = block_excl_scan_p2(s, &tot);
    P2 p{below.a + ex.a, below.b + ex.b};
#pragma unroll
    for (int j = 0; j < SCAN_EPT; ++j) {
        if (i0 + j < count) emit(i0 + j, x[j], p);
        p.a += x[j].a;
        p.b += x[j].b;
    }
}

// The passes over `count` elements; without an `emit` only the grand total.
template <class Val, class Emit>
static void run_tiles(const Val &val, int64_t count, P2 *totals, Grand *grand, Gate gate, const Emit *emit,
                      hipStream_t s)
{
    const int64_t ntiles = (count + SCAN_TILE - 1) / SCAN_TILE;
    const bool self = ntiles <= SELF_TILES && emit;
    hipLaunchKernelGGL(scan_reduce<Val>, dim3((uint32_t)ntiles), dim3(GFR_BLOCK), 0, s, val, count, totals);
    if (!self) hipLaunchKernelGGL(scan_totals, dim3(1), dim3(GFR_BLOCK), 0, s, totals, ntiles, grand);
    if (emit)
        hipLaunchKernelGGL((scan_emit<Val, Emit>), dim3((uint32_t)ntiles), dim3(GFR_BLOCK), 0, s, val, count, totals,
                           ntiles, self, grand, gate, *emit);
    GFR_LAUNCH_CHECK();
}

// ------------------------------------------------------------ advance

struct AdvVal {
    const int32_t *F;
    const int32_t *R;
    int32_t n;
    __device__ bool bad(int64_t i) const { return (uint32_t)F[i] >= (uint32_t)n; }
    __device__ P2 operator()(int64_t i) const
    {
        const int32_t v = F[i];
        if ((uint32_t)v >= (uint32_t)n) return P2{0ull, 0ull};
        const unsigned long long d = (unsigned long long)(R[v + 1] - R[v]);
        return P2{d, d ? 1ull : 0ull};
    }
};

// entries with edges become the queue, tagged with their input item (the
// vertex itself, or the edge it was reached by); part[c] = entry holding edge
// c * CH
struct AdvEmit {
    const int32_t *F;
    const int32_t *T;
    const int32_t *R;
    FrontierQ q;
    __device__ void operator()(int64_t i, P2 x, P2 p) const
    {
        if (!x.a) return;
        const int32_t v = F[i];
        const uint32_t slot = (uint32_t)p.b, off = (uint32_t)p.a, d = (uint32_t)x.a;
        q.v[slot] = T[i];
        q.off[slot] = off;
        q.row[slot] = R[v];
        for (uint32_t c = (off + GATHER_CH - 1) / GATHER_CH; (uint64_t)c * GATHER_CH < (uint64_t)off + d; ++c)
            q.part[c] = (int32_t)slot;
    }
};

// every edge of the queue, written at its offset
__global__ __launch_bounds__(GFR_BLOCK) void advance_emit(FrontierQ q, const Grand *grand, Gate gate, const int32_t *C,
                                                          int32_t *out_src, int32_t *out_edge, int32_t *out_dst)
{
    const Grand g = *grand;
    if (!gate.open(g)) return;
    const uint32_t mf = (uint32_t)g.tot.a, nf = (uint32_t)g.tot.b;
    constexpr uint32_t CH = GATHER_CH;
    __shared__ uint32_t s_off[CH + 1];
    __shared__ int32_t s_row[CH + 1];
    __shared__ int32_t s_v[CH + 1];
    const uint32_t nchunks = (mf + CH - 1) / CH;
    for (uint32_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const uint32_t e0 = c * CH, e1 = min(e0 + CH, mf);
        const int s = q.part[c];
        const int t = (c + 1 < nchunks) ? q.part[c + 1] : (int)nf - 1;
        const int cnt = t - s + 1;
        __syncthreads();
        for (int i = threadIdx.x; i < cnt; i += GFR_BLOCK) {
            s_off[i] = q.off[s + i];
            s_row[i] = q.row[s + i];
            s_v[i] = q.v[s + i];
        }
        __syncthreads();
        for (uint32_t p = e0 + threadIdx.x; p < e1; p += GFR_BLOCK) {
            const int i = upper_index(s_off, 0, cnt - 1, p);
            const int32_t e = s_row[i] + (int32_t)(p - s_off[i]);
            if (out_src) out_src[p] = s_v[i];
            if (out_edge) out_edge[p] = e;
            if (out_dst) out_dst[p] = C[e];
        }
    }
}

// far ends of an edge frontier (-1 for an id outside [0, m))
__global__ void edge_heads(const int32_t *E, int64_t count, const int32_t *C, int32_t m, int32_t *V)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        V[i] = (uint32_t)E[i] < (uint32_t)m ? C[E[i]] : -1;
}

// input list on the device (copied there when it is host memory)
static const int32_t *device_list(const int32_t *list, int64_t count, int32_t *staging, hipStream_t s)
{
    if (is_device_ptr(list)) return list;
    GFR_HIP(hipMemcpyAsync(staging, list, 4ull * count, hipMemcpyHostToDevice, s));
    return staging;
}

// work-groups for one thread per element, at most as many as fit at once
static dim3 list_grid(const Ctx &c, int64_t count)
{
    return dim3((uint32_t)std::min<int64_t>((count + GFR_BLOCK - 1) / GFR_BLOCK, grid_blocks(c, 8)));
}

static Grand grand_back(Ctx &c, const Grand *grand, hipStream_t s, const char *who, const char *what = "vertex")
{
    Grand h;
    read_back(c, grand, sizeof h, s);
    c.waited = true;
    memcpy(&h, c.pinned, sizeof h);
    if (h.bad) fail(GFR_E_INVALID, std::string(who) + ": " + what + " id out of range");
    return h;
}

int64_t run_advance(Ctx &c, Graph &g, const int32_t *frontier, int32_t nf, bool edges, int32_t *out_src,
                    int32_t *out_edge, int32_t *out_dst, int64_t out_cap, hipStream_t s)
{
    const int64_t ntiles = (nf + SCAN_TILE - 1) / SCAN_TILE;
    const int64_t cap = std::min<int64_t>(out_cap, INT32_MAX);
    const size_t nparts = (size_t)(cap / GATHER_CH) + 2;
    c.arena.reserve(2 * al256(4ull * nf) + al256(16ull * ntiles) + al256(sizeof(Grand)) + 3 * al256(4ull * nf) +
                    al256(4 * nparts));
    int32_t *staging = c.arena.take<int32_t>(nf);
    int32_t *heads = c.arena.take<int32_t>(nf);
    P2 *totals = c.arena.take<P2>(ntiles);
    Grand *grand = c.arena.take<Grand>(1);
    FrontierQ q{c.arena.take<int32_t>(nf), c.arena.take<uint32_t>(nf), c.arena.take<int32_t>(nf),
                c.arena.take<int32_t>(nparts)};
    if (nf == 0) return 0;
    const int32_t *R = g.R.as<int32_t>();
    const int32_t *T = device_list(frontier, nf, staging, s), *F = T;   // tags written as out_src; vertices expanded
    if (edges) {
        hipLaunchKernelGGL(edge_heads, list_grid(c, nf), dim3(GFR_BLOCK), 0, s, T, (int64_t)nf, g.C.as<int32_t>(),
                           (int32_t)g.m, heads);
        F = heads;
    }
    const Gate gate{(unsigned long long)cap, ANY};
    const AdvEmit emit{F, T, R, q};
    run_tiles(AdvVal{F, R, g.n}, nf, totals, grand, gate, cap > 0 ? &emit : nullptr, s);   // (no room: the count alone)
    if (cap > 0) {
        const uint32_t most = (uint32_t)std::min<int64_t>(nparts, grid_blocks(c, 4));
        hipLaunchKernelGGL(advance_emit, dim3(most), dim3(GFR_BLOCK), 0, s, q, grand, gate, g.C.as<int32_t>(), out_src,
                           out_edge, out_dst);
    }
    GFR_LAUNCH_CHECK();
    const Grand h = grand_back(c, grand, s, edges ? "advance_edges" : "advance", edges ? "edge" : "vertex");
    const int64_t total = (int64_t)h.tot.a;
    if (total > out_cap || total > INT32_MAX) return total;   // nothing was written; the caller reports the capacity error
    c.stats.v["edges"] = (double)total;
    c.stats.v["entries_with_edges"] = (double)h.tot.b;
    return total;
}

// ------------------------------------------------------------- filter

__global__ void mark_items(const int32_t *items, int64_t count, int32_t n, const uint8_t *exclude, uint8_t *mark,
                           uint32_t *bad)
{
    bool wrong = false;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = items[i];
        if ((uint32_t)v >= (uint32_t)n) wrong = true;
        else if (!exclude || !exclude[v]) mark[v] = 1;
    }
    if (wrong) *bad = 1u;
}

struct MarkVal {
    const uint8_t *mark;
    const uint32_t *marked_bad;
    __device__ bool bad(int64_t i) const { return i == 0 && *marked_bad; }   // noted where the items were read
    __device__ P2 operator()(int64_t i) const { return P2{0ull, mark[i] ? 1ull : 0ull}; }
};

struct ListEmit {
    int32_t *out;
    __device__ void operator()(int64_t i, P2 x, P2 p) const
    {
        if (x.b) out[p.b] = (int32_t)i;
    }
};

int64_t run_filter(Ctx &c, Graph &g, const int32_t *items, int64_t count, const uint8_t *exclude, int32_t *out,
                   int64_t out_cap, hipStream_t s)
{
    const int32_t n = g.n;
    const int64_t ntiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    c.arena.reserve(al256(4ull * count) + al256(16ull * ntiles) + al256(sizeof(Grand)) + al256(4) +
                    al256(4ull * ((n + 3) / 4)) + al256(n));
    int32_t *staging = c.arena.take<int32_t>(count);
    P2 *totals = c.arena.take<P2>(ntiles);
    Grand *grand = c.arena.take<Grand>(1);
    uint32_t *bad = c.arena.take<uint32_t>(1);
    uint8_t *mark = c.arena.take<uint8_t>(4ull * ((n + 3) / 4));
    if (exclude && !is_device_ptr(exclude)) {
        uint8_t *excl_dev = c.arena.take<uint8_t>(n);
        GFR_HIP(hipMemcpyAsync(excl_dev, exclude, (size_t)n, hipMemcpyHostToDevice, s));
        exclude = excl_dev;
    }
    // (a copy from pageable memory waits for what is queued before it, so it comes first)
    const int32_t *X = count > 0 ? device_list(items, count, staging, s) : nullptr;
    Fills().add(mark, 0u, (n + 3) / 4).add(bad, 0u, 1).run(s);
    if (count > 0)
        hipLaunchKernelGGL(mark_items, list_grid(c, count), dim3(GFR_BLOCK), 0, s, X, count, n, exclude, mark,
                           bad);
    const ListEmit emit{out};
    run_tiles(MarkVal{mark, bad}, n, totals, grand, Gate{ANY, (unsigned long long)out_cap}, &emit, s);
    const int64_t kept = (int64_t)grand_back(c, grand, s, "filter").tot.b;
    if (kept > out_cap) return kept;   // nothing was written; the caller reports the capacity error
    c.stats.v["kept"] = (double)kept;
    return kept;
}

// ------------------------------------------------------------- scan

struct ScanVal {
    const uint32_t *x;
    __device__ bool bad(int64_t) const { return false; }
    __device__ P2 operator()(int64_t i) const { return P2{(unsigned long long)x[i], 0ull}; }
};

struct ScanEmit {
    unsigned long long *out;
    __device__ void operator()(int64_t i, P2, P2 p) const { out[i] = p.a; }
};

uint64_t run_scan(Ctx &c, const uint32_t *in, int64_t count, unsigned long long *out, hipStream_t s)
{
    const int64_t ntiles = (count + SCAN_TILE - 1) / SCAN_TILE;
    c.arena.reserve(al256(4ull * count) + al256(16ull * ntiles) + al256(sizeof(Grand)));
    uint32_t *staging = c.arena.take<uint32_t>(count);
    P2 *totals = c.arena.take<P2>(ntiles);
    Grand *grand = c.arena.take<Grand>(1);
    if (count == 0) return 0;
    const uint32_t *X = (const uint32_t *)device_list((const int32_t *)in, count, (int32_t *)staging, s);
    const ScanEmit emit{out};
    run_tiles(ScanVal{X}, count, totals, grand, Gate{ANY, ANY}, &emit, s);
    return grand_back(c, grand, s, "scan").tot.a;
}

// ------------------------------------------------------------- split

struct SplitVal {
    const int32_t *X;
    const uint32_t *dist;
    uint32_t thr;
    int32_t n;
    __device__ bool bad(int64_t i) const { return (uint32_t)X[i] >= (uint32_t)n; }
    __device__ P2 operator()(int64_t i) const
    {
        if (bad(i)) return P2{0ull, 0ull};
        const bool nr = dist[X[i]] < thr;
        return P2{nr ? 1ull : 0ull, nr ? 0ull : 1ull};
    }
};

struct SplitEmit {
    const int32_t *X;
    int32_t *near, *far;
    __device__ void operator()(int64_t i, P2 x, P2 p) const
    {
        if (x.a) near[p.a] = X[i];
        else far[p.b] = X[i];
    }
};

void run_split(Ctx &c, Graph &g, const int32_t *items, int64_t count, const uint32_t *dist, uint32_t threshold,
               int32_t *near, int32_t *far, int64_t out_cap, int64_t *n_near, int64_t *n_far, hipStream_t s)
{
    const int32_t n = g.n;
    const int64_t ntiles = (count + SCAN_TILE - 1) / SCAN_TILE;
    c.arena.reserve(al256(4ull * count) + al256(16ull * ntiles) + al256(sizeof(Grand)) + al256(4ull * n));
    int32_t *staging = c.arena.take<int32_t>(count);
    P2 *totals = c.arena.take<P2>(ntiles);
    Grand *grand = c.arena.take<Grand>(1);
    uint32_t *dist_dev = c.arena.take<uint32_t>(n);
    *n_near = *n_far = 0;
    if (count == 0) return;
    const int32_t *X = device_list(items, count, staging, s);
    const uint32_t *D = dist;
    if (!is_device_ptr(dist)) {
        GFR_HIP(hipMemcpyAsync(dist_dev, dist, 4ull * n, hipMemcpyHostToDevice, s));
        D = dist_dev;
    }
    const SplitEmit emit{X, near, far};
    run_tiles(SplitVal{X, D, threshold, n}, count, totals, grand,
              Gate{(unsigned long long)out_cap, (unsigned long long)out_cap}, &emit, s);
    const Grand h = grand_back(c, grand, s, "split");
    *n_near = (int64_t)h.tot.a;
    *n_far = (int64_t)h.tot.b;   // (nothing was written when either exceeds out_cap)
}

}  // namespace gfr
