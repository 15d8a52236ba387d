// bfs.hip -- single-source BFS: level-synchronous advance + filter with a
// per-level push/pull choice (Sec. 4.5 "Push vs. pull traversal", Sec. 5.1).
//
// Every level is two launches:
//   bfs_level   the advance.  Push: the frontier queue carries the exclusive
//               scan of its degrees and a chunk index, so every work-group
//               takes an equal slice of the frontier's edges (load-balanced
//               partitioning, Sec. 4.4); each edge tests the visited bitmap
//               and, for an unvisited neighbour not yet marked, writes its
//               depth and a mark byte with plain stores.  This is the
//               idempotent advance of Sec. 4.5: concurrent discoverers write
//               the same values, and the compaction removes the duplicates.
//               (With bfs.dedup = 0 the neighbour is first claimed with an
//               atomicOr on the visited bitmap, the non-idempotent form.)
//               Pull: every unvisited vertex scans its list until it meets a
//               vertex of the current frontier bitmap; a lane takes the first
//               entries of its vertex, then quarter waves the long lists left.
//               Either way the new frontier is a byte array of marks.
//   compact     the filter: the marks become the next queue in vertex order
//               and the next frontier bitmap, visited is updated (compact.h),
//               and the last work-group runs the level control:
//               stop on an empty frontier, otherwise choose push or pull from
//               the frontier's edge count against the unvisited vertices'
//               (the rule of Sec. 4.5, with tunable ratios alpha and beta).
// The control state lives in device memory, so the host enqueues levels
// speculatively and only reads one word back every few levels.
//
// On mesh-like graphs (small, even degrees, long diameters) the frontier is
// kept as mark bytes only, with one launch per level (bfs_bitmap_level): each
// thread owns a run of vertices, consumes their marks of the current level,
// stores the depths of those not yet visited and lists them in LDS; the
// work-group expands the list and marks unvisited neighbours for the next
// level, with plain idempotent stores (Sec. 4.5).  There is no queue and no
// compaction: on such graphs a level's cost is the chain of memory round trips
// of its launches, and this halves the number of launches and drops the
// compaction's scan and look-back.  Each work-group records whether it held a
// vertex; a later launch's first work-group reads those flags and ends the
// traversal when all are zero.
#include <algorithm>

#include "compact.h"
#include "device.h"
#include "engine.h"

namespace gfr {

enum : uint32_t { DIR_PUSH = 0, DIR_PULL = 1, DIR_DONE = 2 };

struct BfsCtl {
    uint32_t dir;       // DIR_* of the current level (first word: read back by the host)
    int32_t level;      // depth of the current frontier
    uint32_t nf, mf;    // entries / edges of the current queue
    unsigned long long mu;  // edges incident to unvisited vertices
    uint32_t nu;        // unvisited vertices
    uint32_t force;     // 0 auto, 1 push only, 2 pull only
    uint32_t dedup;     // 0 atomic claim, 1 idempotent
    float alpha, beta;
    uint32_t parity;    // status-buffer parity of the compaction
    uint32_t err;       // compaction look-back gave up (never expected)
    uint32_t ticket;    // of the compaction
    uint32_t push_levels, pull_levels;
    // traffic model counters (summed over levels)
    unsigned long long push_entries, push_edges, push_new;
    unsigned long long pull_unvisited, pull_inspected, pull_new;
};

struct BfsArgs {
    const int32_t *R;
    const int32_t *C;
    int32_t n;
    uint32_t nwords;
    int32_t *depth;
    uint32_t *vis;        // visited bitmap (updated by the compaction)
    uint32_t *fb;         // current frontier bitmap (written by the compaction)
    uint8_t *mark;        // next-frontier marks, one byte per vertex
    FrontierQ q;
    const int32_t *likely;   // first neighbour to probe in a pull level (-1: no edges), or null
    uint32_t *part_insp;   // per work-group edges inspected by a pull level
    BfsCtl *ctl;
    uint32_t mapping;        // push work mapping: 0 by frontier size, 1 edge chunks, 2 per-vertex groups
    uint32_t twc_threshold;  // mapping 0: per-vertex groups below this many frontier vertices
};

// One push edge of BFS level L: test the visited bit, claim (or, idempotent,
// just write) an unvisited target's depth and next-frontier mark.
__device__ __forceinline__ void bfs_push_edge(const BfsArgs &a, int32_t v, int32_t L, bool idem)
{
    const uint32_t bit = 1u << (v & 31);
    uint32_t *w = a.vis + (v >> 5);
    if (!(*w & bit) && !a.mark[v]) {
        if (idem || !(atomicOr(w, bit) & bit)) {
            a.depth[v] = L + 1;
            a.mark[v] = 1;
        }
    }
}

// The per-vertex mapping of Sec. 4.4 (per-CTA / per-warp coarse-grained,
// then the fine-grained strategy for the rest): each work-group takes
// GFR_BLOCK frontier vertices, one per thread.  Lists of at least GFR_BLOCK
// edges are taken one at a time by the whole work-group (their owners compete
// for it through an LDS word), then lists of at least 64 edges one at a time
// by the owner's wave.  The remaining short lists are processed by the whole
// work-group together: their sizes are scanned, the list offsets sit in LDS,
// and each thread takes every GFR_BLOCK-th of their edges, finding its list
// by binary search (the cooperative fine-grained form of Sec. 4.4).
__device__ void bfs_push_twc(const BfsArgs &a, const FrontierQ &q, uint32_t nf, uint32_t mf, int32_t L, bool idem)
{
    __shared__ int32_t s_owner, s_row, s_deg;
    __shared__ uint32_t s_soff[GFR_BLOCK + 1];
    __shared__ int32_t s_srow[GFR_BLOCK];
    __shared__ uint32_t s_wsum[GFR_WAVES];
    const int lane = lane_id(), wave = threadIdx.x / 64;
    for (uint32_t base = blockIdx.x * GFR_BLOCK; base < nf; base += gridDim.x * GFR_BLOCK) {
        const uint32_t i = base + threadIdx.x;
        int32_t row = 0, deg = 0;
        if (i < nf) {
            row = q.row[i];
            deg = (int32_t)((i + 1 < nf ? q.off[i + 1] : mf) - q.off[i]);
        }
        for (;;) {   // work-group lists
            if (threadIdx.x == 0) s_owner = -1;
            __syncthreads();
            if (deg >= GFR_BLOCK) s_owner = (int32_t)threadIdx.x;   // one of the writers wins
            __syncthreads();
            const int32_t owner = s_owner;
            if (owner < 0) break;
            if ((int32_t)threadIdx.x == owner) {
                s_row = row;
                s_deg = deg;
                deg = 0;
            }
            __syncthreads();
            const int32_t r0 = s_row, d0 = s_deg;
            for (int32_t k = (int32_t)threadIdx.x; k < d0; k += GFR_BLOCK) bfs_push_edge(a, a.C[r0 + k], L, idem);
            __syncthreads();   // s_row / s_deg are rewritten by the next owner
        }
        for (;;) {   // wave lists
            const uint64_t want = ballot(deg >= 64);
            if (!want) break;
            const int src = __ffsll((unsigned long long)want) - 1;
            const int32_t r0 = __builtin_amdgcn_readlane(row, src), d0 = __builtin_amdgcn_readlane(deg, src);
            if (lane == src) deg = 0;
            for (int32_t k = lane; k < d0; k += 64) bfs_push_edge(a, a.C[r0 + k], L, idem);
        }
        // short lists, the whole work-group over their concatenated edges
        const uint32_t incl = wave_incl_scan((uint32_t)deg);
        if (lane == 63) s_wsum[wave] = incl;
        __syncthreads();
        uint32_t wbase = 0, total = 0;
        for (int k = 0; k < GFR_WAVES; ++k) {
            if (k < wave) wbase += s_wsum[k];
            total += s_wsum[k];
        }
        s_soff[threadIdx.x] = wbase + incl - (uint32_t)deg;
        s_srow[threadIdx.x] = row;
        if (threadIdx.x == 0) s_soff[GFR_BLOCK] = total;
        __syncthreads();
        for (uint32_t e = threadIdx.x; e < total; e += GFR_BLOCK) {
            const int j = upper_index(s_soff, 0, GFR_BLOCK - 1, e);   // lists of size 0 share offsets: the last wins
            bfs_push_edge(a, a.C[s_srow[j] + (int32_t)(e - s_soff[j])], L, idem);
        }
        __syncthreads();   // LDS is reused by the next slice
    }
}

// What holds a pull level up is the line of C, somewhere in memory, that each
// unvisited vertex reads only to find that one of its first neighbours is in the
// frontier, and the lane that scans a list of hundreds by itself.  On scale-free
// graphs the neighbour of the largest degree is in the frontier more often than
// any other, so its id is kept in an array of its own, made when the graph is
// loaded and read in order: on R-MAT with 524,288 vertices and 15.5 M entries,
// at the level that finds 68 % of the unvisited vertices with edges, it is a
// frontier vertex for 62 %, the first of the list for 50 %.  Lists that a lane
// has not settled after PULL_STEPS steps go to quarter waves.  R-MAT with 4 M
// vertices, the three pull levels: 112, 27 and 14 us as it was, 87, 27 and 14
// with the quarter waves, 63, 19 and 12 with the array as well, 61, 17 and 10
// with the next vertices' words fetched ahead.  (The first LK_MAX neighbours are
// looked at: hubs are hardly ever unvisited by then.)
constexpr int LK_LANES = 16, LK_MAX = 64;
constexpr int PULL_STEPS = 2;   // of 4 probes (1 and 3: the fat level 64 and 63 us, 61 with 2)
// Below 8 M entries C is in the L2s, and the calls are no faster with the array
// (524,288 vertices and 4 M entries 156 / 157 us; 2 M and 63 M 199 / 190).
constexpr int64_t LK_MIN_EDGES = 1 << 23;

__global__ __launch_bounds__(GFR_BLOCK) void likely_kernel(const int32_t *R, const int32_t *C, int32_t n,
                                                           int32_t *likely)
{
    const int32_t lane = (int32_t)(threadIdx.x % LK_LANES);
    const uint32_t groups = gridDim.x * (GFR_BLOCK / LK_LANES);
    for (uint32_t v = (blockIdx.x * GFR_BLOCK + threadIdx.x) / LK_LANES; v < (uint32_t)n; v += groups) {
        const uint32_t r0 = (uint32_t)R[v], r1 = head_end(r0, (uint32_t)R[v + 1], LK_MAX);
        int32_t deg = 0, best = -1;
        for (uint32_t e = r0 + (uint32_t)lane; e < r1; e += LK_LANES) {
            const int32_t u = C[e], d = R[u + 1] - R[u];
            if (d > deg) {
                deg = d;
                best = u;
            }
        }
#pragma unroll
        for (int k = LK_LANES / 2; k >= 1; k >>= 1) {
            const int32_t od = __shfl_xor(deg, k, LK_LANES), ob = __shfl_xor(best, k, LK_LANES);
            if (od > deg) {
                deg = od;
                best = ob;
            }
        }
        // a directed edge may lead to a vertex without edges: any neighbour does then
        if (lane == 0) likely[v] = best >= 0 || r1 == r0 ? best : C[r0];
    }
}

void likely_neighbours(Ctx &c, Graph &g, hipStream_t s)
{
    if (g.cls == GRAPH_MESH || g.m < LK_MIN_EDGES) return;
    try {
        g.likely.alloc(4ull * g.n);
    } catch (const Error &e) {
        if (e.code != GFR_E_OOM) throw;
        (void)hipGetLastError();   // the levels then read the lists
        return;
    }
    g.bytes += g.likely.bytes;
    hipLaunchKernelGGL(likely_kernel, dim3(grid_blocks(c, 8)), dim3(GFR_BLOCK), 0, s, g.R.as<int32_t>(),
                       g.C.as<int32_t>(), g.n, g.likely.as<int32_t>());
    GFR_LAUNCH_CHECK();
}

template <int CH>
__global__ __launch_bounds__(GFR_BLOCK) void bfs_level(BfsArgs a)
{
    BfsCtl *ctl = a.ctl;
    const uint32_t dir = ctl->dir;
    if (dir == DIR_DONE) return;
    const int32_t L = ctl->level;

    if (dir == DIR_PUSH) {
        __shared__ uint32_t s_off[CH + 1];
        __shared__ int32_t s_row[CH + 1];
        const uint32_t mf = ctl->mf, nf = ctl->nf;
        const bool idem = ctl->dedup != 0;
        const FrontierQ q = a.q;
        // Sec. 4.4's hybrid: per-vertex groups for frontiers below the
        // threshold, equal edge chunks (load-balanced partitioning) above it
        if (a.mapping == 2 || (a.mapping == 0 && nf < a.twc_threshold)) {
            bfs_push_twc(a, q, nf, mf, L, idem);
            return;
        }
        const uint32_t nchunks = (mf + CH - 1) / CH;
        for (uint32_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
            const uint32_t e0 = c * CH;
            const uint32_t e1 = min(e0 + (uint32_t)CH, mf);
            const int s = q.part[c];
            const int t = (c + 1 < nchunks) ? q.part[c + 1] : (int)nf - 1;
            const int cnt = t - s + 1;
            __syncthreads();
            for (int i = threadIdx.x; i < cnt; i += GFR_BLOCK) {
                s_off[i] = q.off[s + i];
                s_row[i] = q.row[s + i];
            }
            __syncthreads();
            // each thread takes every GFR_BLOCK-th edge of the chunk: all its
            // column loads are issued first, then all visited-word probes,
            // then the tests (an edge past the chunk end repeats the chunk's
            // first edge and is masked)
            constexpr int PER = CH / GFR_BLOCK;
            int32_t vv[PER];
            uint32_t vw[PER];
            bool ok[PER];
#pragma unroll
            for (int p = 0; p < PER; ++p) {
                const uint32_t e = e0 + p * GFR_BLOCK + threadIdx.x;
                ok[p] = e < e1;
                const uint32_t ec = ok[p] ? e : e0;
                const int i = upper_index(s_off, 0, cnt - 1, ec);
                vv[p] = a.C[s_row[i] + (int32_t)(ec - s_off[i])];
            }
#pragma unroll
            for (int p = 0; p < PER; ++p) vw[p] = a.vis[vv[p] >> 5];
#pragma unroll
            for (int p = 0; p < PER; ++p) {
                const int32_t v = vv[p];
                const uint32_t bit = 1u << (v & 31);
                if (ok[p] && !(vw[p] & bit) && !a.mark[v]) {
                    if (idem || !(atomicOr(a.vis + (v >> 5), bit) & bit)) {
                        a.depth[v] = L + 1;
                        a.mark[v] = 1;
                    }
                }
            }
        }
    } else {
        const uint32_t waves = gridDim.x * GFR_WAVES;
        const int lane = lane_id();
        uint32_t insp = 0;
        // (the next 64 vertices' words, offsets and likely neighbours are
        // fetched beside these ones' probes)
        const uint32_t end = ((uint32_t)a.n + 63u) / 64u;
        uint32_t grp = blockIdx.x * GFR_WAVES + threadIdx.x / 64;
        uint32_t visw_n = 0;
        int32_t u_n = 0;
        uint32_t e_n = 0, re_n = 0;
        const auto fetch = [&](uint32_t gr) {
            if (gr >= end) return;
            const uint32_t x = min(gr * 64u + (uint32_t)lane, (uint32_t)a.n - 1u);
            visw_n = a.vis[gr * 2u + (uint32_t)(lane >> 5)];
            u_n = a.likely ? a.likely[x] : 0;
            e_n = (uint32_t)a.R[x];
            re_n = (uint32_t)a.R[x + 1u];
        };
        fetch(grp);
        for (; grp < end; grp += waves) {
            const int32_t v = (int32_t)(grp * 64u) + lane;
            const bool open = v < a.n && !(visw_n & (1u << (v & 31)));
            const int32_t u = u_n;
            uint32_t e = open ? e_n : 0u, re = open ? re_n : 0u;
            fetch(grp + waves);
            bool found = false;
            if (a.likely && e < re) {
                ++insp;
                found = (a.fb[u >> 5] >> (u & 31)) & 1u;
            }
            // a lane's first entries, four independent probes per step
            for (int step = 0; step < PULL_STEPS && e < re && !found; ++step) {
                const uint32_t k = min(4u, re - e);
                int32_t u[4];
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) u[j] = a.C[j < k ? e + j : e];
                uint32_t hit = 0;
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) hit |= (j < k) ? (a.fb[u[j] >> 5] >> (u[j] & 31)) & 1u : 0u;
                insp += k;
                found = hit != 0;
                e += 4;
            }
            // the rest of the long lists, four at a time by a quarter of the wave each
            uint64_t todo = ballot(e < re && !found);
            while (todo) {
                uint64_t mine = todo;
                for (int j = 0; j < lane / 16; ++j) mine &= mine - 1;
                const int owner = mine ? __ffsll((unsigned long long)mine) - 1 : 0;
                uint32_t p = shfl_u32(e, owner), end = shfl_u32(re, owner);   // (the owner may sit in any quarter)
                if (!mine) end = p;
                bool hit = false;
                while (p < end && !hit) {
                    const uint32_t i = (uint32_t)lane % 16u;
                    const int32_t u0 = a.C[entry_or_last(p, i, end)], u1 = a.C[entry_or_last(p, i + 16u, end)];
                    const uint32_t f0 = a.fb[u0 >> 5] >> (u0 & 31), f1 = a.fb[u1 >> 5] >> (u1 & 31);
                    hit = ((ballot((f0 | f1) & 1u) >> (lane & 48)) & 0xFFFFull) != 0;
                    if (lane % 16 == 0) insp += min(32u, end - p);
                    p += 32;
                }
                const uint64_t hits = ballot(hit);
                if ((todo >> lane) & 1ull) {
                    const int rank = __popcll(todo & ((1ull << lane) - 1ull));
                    if (rank < 4) found = (hits >> (16 * rank)) & 1ull;
                }
                for (int j = 0; j < 4; ++j) todo &= todo - 1;
            }
            if (found) {
                a.depth[v] = L + 1;
                a.mark[v] = 1;
            }
        }
        // per-group partial (plain store, summed by the level control)
        __shared__ uint32_t s_insp[GFR_WAVES];
        const uint32_t tot = wave_sum_u32(insp);
        if (lane == 0) s_insp[threadIdx.x / 64] = tot;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t t = 0;
            for (int i = 0; i < GFR_WAVES; ++i) t += s_insp[i];
            a.part_insp[blockIdx.x] = t;
        }
    }
}

// Filter + level control for the compaction kernel.
struct BfsMarks {
    BfsArgs a;
    uint32_t nparts;   // work-groups of bfs_level (entries of part_insp)

    __device__ bool skip() const { return a.ctl->dir == DIR_DONE; }
    __device__ uint32_t mask(uint32_t w) const
    {
        const uint32_t m = marks_to_mask(a.mark + 32ull * w);
        if (m) {
            clear_marks(a.mark + 32ull * w);
            a.vis[w] |= m;
        }
        a.fb[w] = m;
        return m;
    }
    __device__ void partial(uint32_t) {}
    __device__ void control(uint32_t nf2, uint32_t mf2) const
    {
        BfsCtl *ctl = a.ctl;
        const uint32_t dir = ctl->dir;
        uint32_t insp = 0;
        if (dir == DIR_PULL) {
            for (uint32_t i = threadIdx.x; i < nparts; i += GFR_BLOCK) insp += a.part_insp[i];
            __shared__ uint32_t s[GFR_WAVES];
            insp = wave_sum_u32(insp);
            if (lane_id() == 0) s[threadIdx.x / 64] = insp;
            __syncthreads();
            insp = 0;
            for (int i = 0; i < GFR_WAVES; ++i) insp += s[i];
        }
        if (threadIdx.x != 0) return;
        if (dir == DIR_PUSH) {
            ctl->push_levels += 1;
            ctl->push_entries += ctl->nf;
            ctl->push_edges += ctl->mf;
            ctl->push_new += nf2;
        } else {
            ctl->pull_levels += 1;
            ctl->pull_unvisited += ctl->nu;
            ctl->pull_inspected += insp;
            ctl->pull_new += nf2;
        }
        ctl->nu -= nf2;
        ctl->mu -= mf2;
        uint32_t nd;
        if (nf2 == 0) nd = DIR_DONE;
        else if (ctl->force == 1) nd = DIR_PUSH;
        else if (ctl->force == 2) nd = DIR_PULL;
        else if (dir == DIR_PUSH)
            nd = ((double)mf2 > (double)ctl->mu / ctl->alpha && nf2 > ctl->nf) ? DIR_PULL : DIR_PUSH;
        else
            nd = ((double)nf2 < (double)a.n / ctl->beta && nf2 < ctl->nf) ? DIR_PUSH : DIR_PULL;
        ctl->nf = nf2;
        ctl->mf = mf2;
        ctl->level += 1;
        ctl->parity ^= 1u;
        ctl->dir = nd;
    }
};

// the queue of the source alone, and the control block (one work-group)
struct BfsFirst {
    BfsArgs a;
    int32_t src;
    uint32_t chunk, force, dedup;
    float alpha, beta;
    unsigned long long m;
    __device__ void operator()() const
    {
        const int32_t rs = a.R[src], deg = a.R[src + 1] - rs;
        if (threadIdx.x == 0) {
            BfsCtl *ctl = a.ctl;
            a.q.v[0] = src;
            a.q.off[0] = 0;
            a.q.row[0] = rs;
            ctl->mu = m - (unsigned long long)deg;
            ctl->nf = 1;
            ctl->mf = (uint32_t)deg;
            ctl->level = 0;
            ctl->nu = (uint32_t)a.n - 1u;
            ctl->force = force;
            ctl->dedup = dedup;
            ctl->alpha = alpha;
            ctl->beta = beta;
            ctl->parity = 0;
            ctl->err = 0;
            ctl->ticket = 0;
            ctl->push_levels = ctl->pull_levels = 0;
            ctl->push_entries = ctl->push_edges = ctl->push_new = 0ull;
            ctl->pull_unvisited = ctl->pull_inspected = ctl->pull_new = 0ull;
            ctl->dir = deg == 0 ? DIR_DONE : (force == 2 ? DIR_PULL : DIR_PUSH);
        }
        for (uint32_t c = threadIdx.x; (uint64_t)c * chunk < (uint64_t)deg; c += blockDim.x) a.q.part[c] = 0;
    }
};

// ------------------------------------------------------------ mark-byte levels
// What bounds a level is its chain of dependent memory round trips (marks, row
// offsets, columns, depths), each about a microsecond, and the launch; so a
// level should walk that chain once.  A work-group takes one span of
// BM_BLOCK * VPT vertices: VPT is chosen so that all spans of the graph are
// resident at once (up to 2^24 vertices), and a span's marked vertices, listed
// in LDS as 16-bit offsets, usually fit one turn of the threads.  Spans keep
// the expansion in vertex order, which a mesh rewards: neighbouring frontier
// vertices share the lines of their rows and depths.  (A list of the frontier
// in discovery order was slower, 85 us against 20 for levels of 600 K
// vertices, for that reason.)
//
// On the 4096^2 lattice (139 levels of 120 K vertices on average) a level took
// 19.5 us in two turns of 4 KB spans that probed and stored depth[] by edge.  It
// takes 4 to 9 us while the frontier is thin and 43 us at its widest (600 K
// vertices: about 200 MB of distinct lines, 4.6 TB/s), 13 us on average.
//
// The first levels, up to BM_SOLO vertices each, are run by one work-group in
// one launch with the frontier in LDS (38 levels in 167 us there).
constexpr int BM_BLOCK = 512;
constexpr int BM_SOLO_BLOCK = 1024;
constexpr uint32_t BM_SOLO = BM_SOLO_BLOCK;      // widest level that one work-group runs
constexpr uint32_t BM_SOLO_LIST = 4096;          // discoveries it can list; more are marked at once
constexpr int32_t BM_SOLO_LEVELS = 1 << 14;      // most levels in one launch

struct BmArgs {
    const int32_t *R;
    const int32_t *C;
    int32_t n;
    int32_t *depth;
    uint8_t *mk[2];      // mark bytes of the frontier, by level parity (n rounded up to 64 bytes)
    uint32_t *vis;       // visited bitmap (null: depth[] alone says what is visited)
    uint32_t *flags;     // [2][gridDim]: did the work-group hold a vertex of the level, by level parity
    BfsCtl *ctl;
};

// Levels 0, 1, ... while they hold at most BM_SOLO vertices (one work-group).
// A discovery is claimed with an atomicOr on its visited bit, so the list
// holds every vertex once.  Leaves ctl->level at the first level not expanded,
// whose vertices it marks, unvisited as the level kernel expects them;
// DIR_DONE if there is none.
__global__ __launch_bounds__(BM_SOLO_BLOCK) void bfs_bitmap_head(BmArgs a, int32_t src)
{
    __shared__ int32_t s_cur[BM_SOLO], s_new[BM_SOLO_LIST];
    __shared__ uint32_t s_cnt;
    uint32_t cnt = 1;
    if (threadIdx.x == 0) {
        a.depth[src] = 0;
        atomicOr(a.vis + (src >> 5), 1u << (src & 31));
        s_cur[0] = src;
        s_cnt = 0;
    }
    __syncthreads();
    int32_t L = 0;
    for (;;) {
        if (threadIdx.x < cnt) {
            const int32_t v = s_cur[threadIdx.x];
            const uint32_t e1 = (uint32_t)a.R[v + 1];
            for (uint32_t e = (uint32_t)a.R[v]; e < e1; e += 8) {
                int32_t u[8];
                uint32_t old[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) u[k] = a.C[entry_or_last(e, k, e1)];
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (e + k < e1) old[k] = atomicOr(a.vis + (u[k] >> 5), 1u << (u[k] & 31));
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    if (e + k < e1 && !(old[k] >> (u[k] & 31) & 1u)) {
                        a.depth[u[k]] = L + 1;
                        const uint32_t i = atomicAdd(&s_cnt, 1u);
                        if (i < BM_SOLO_LIST) {
                            s_new[i] = u[k];
                        } else {   // too wide for the head: handed over at once
                            atomicAnd(a.vis + (u[k] >> 5), ~(1u << (u[k] & 31)));
                            a.mk[(L & 1) ^ 1][u[k]] = 1;
                        }
                    }
                }
            }
        }
        __syncthreads();
        cnt = s_cnt;
        ++L;
        if (cnt == 0 || cnt > BM_SOLO || L == BM_SOLO_LEVELS) break;
        __syncthreads();
        if (threadIdx.x == 0) s_cnt = 0;
        if (threadIdx.x < cnt) s_cur[threadIdx.x] = s_new[threadIdx.x];
        __syncthreads();
    }
    for (uint32_t i = threadIdx.x; i < min(cnt, BM_SOLO_LIST); i += BM_SOLO_BLOCK) {
        const int32_t u = s_new[i];
        atomicAnd(a.vis + (u >> 5), ~(1u << (u & 31)));
        a.mk[L & 1][u] = 1;
    }
    if (threadIdx.x == 0) {
        BfsCtl *ctl = a.ctl;
        ctl->dir = cnt > 0 ? DIR_PUSH : DIR_DONE;
        ctl->level = L;
        ctl->err = 0;
        ctl->push_levels = (uint32_t)L;
        ctl->pull_levels = 0;
        ctl->push_entries = ctl->push_edges = ctl->push_new = 0ull;
        ctl->pull_unvisited = ctl->pull_inspected = ctl->pull_new = 0ull;
        ctl->nf = (uint32_t)L;   // the head's levels
    }
}

// without the head: the source alone is marked
__global__ void bfs_bitmap_init(BmArgs a, int32_t src)
{
    BfsCtl *ctl = a.ctl;
    a.mk[0][src] = 1;
    ctl->dir = DIR_PUSH;
    ctl->level = 0;
    ctl->err = 0;
    ctl->push_levels = ctl->pull_levels = 0;
    ctl->push_entries = ctl->push_edges = ctl->push_new = 0ull;
    ctl->pull_unvisited = ctl->pull_inspected = ctl->pull_new = 0ull;
    ctl->nf = 0;
}

// One level per launch: launch i runs level ctl->nf + i.  VIS: probe and keep
// the visited bitmap.  A thread owns VPT consecutive vertices: it alone
// consumes their marks, drops those already visited, sets their visited bits
// and stores their depths.  An edge therefore only probes one bit (the bitmap
// of 2^24 vertices is 2 MB and stays in L2; depth[] is 64 MB) and stores one
// mark.  A probe that misses the bit of a vertex of the same level, which its
// owner is just setting, leaves a mark that the owner drops in the next launch.
template <int BLOCK, int VPT, bool VIS>
__global__ __launch_bounds__(BLOCK) void bfs_bitmap_level(BmArgs a, int32_t launch)
{
    static_assert((VPT == 16 || VPT == 32) && BLOCK * VPT <= 65536, "16-bit offsets in a span");
    constexpr int VEC = VPT / 16;
    constexpr int SPAN = BLOCK * VPT;
    __shared__ uint16_t s_v[SPAN];
    __shared__ uint32_t s_cnt;
    BfsCtl *ctl = a.ctl;
    const uint32_t G = gridDim.x;
    if (ctl->dir == DIR_DONE) return;
    const int32_t L = (int32_t)ctl->nf + launch;
    uint8_t *cur = a.mk[L & 1];
    uint8_t *nxt = a.mk[(L & 1) ^ 1];
    int found = 0;
    const size_t nown = ((size_t)a.n + VPT - 1) / VPT;   // owners (the mark bytes are padded to whole ones)
    for (size_t span = blockIdx.x; span * BLOCK < nown; span += G) {
        if (threadIdx.x == 0) s_cnt = 0;
        __syncthreads();
        const size_t own = span * BLOCK + threadIdx.x;
        uint4 w[VEC];
#pragma unroll
        for (int j = 0; j < VEC; ++j)
            w[j] = own < nown ? *(const uint4 *)(cur + own * VPT + 16 * j) : make_uint4(0u, 0u, 0u, 0u);
        uint32_t m = 0;
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            if ((w[j].x | w[j].y | w[j].z | w[j].w) == 0u) continue;
            *(uint4 *)(cur + own * VPT + 16 * j) = make_uint4(0u, 0u, 0u, 0u);   // consumed
            const uint32_t ws[4] = {w[j].x, w[j].y, w[j].z, w[j].w};
#pragma unroll
            for (int k = 0; k < 4; ++k)
                m |= ((ws[k] & 0x01010101u) * 0x00204081u >> 21 & 0xFu) << (16 * j + 4 * k);
        }
        const int32_t v0 = (int32_t)(span * SPAN);
        if (m) {
            if (VIS) {
                if (VPT == 32) {
                    const uint32_t old = a.vis[own];
                    m &= ~old;
                    if (m) a.vis[own] = old | m;
                } else {
                    uint16_t *vw = (uint16_t *)a.vis + own;
                    const uint32_t old = *vw;
                    m &= ~old;
                    if (m) *vw = (uint16_t)(old | m);
                }
            }
            uint32_t i = m ? atomicAdd(&s_cnt, (uint32_t)__popc(m)) : 0u;
            while (m) {
                const int b = __ffs(m) - 1;
                m &= m - 1;
                s_v[i++] = (uint16_t)(threadIdx.x * VPT + b);
            }
        }
        __syncthreads();
        const uint32_t cnt = s_cnt;   // at most SPAN
        for (uint32_t i = threadIdx.x; i < cnt; i += BLOCK) {
            const int32_t v = v0 + s_v[i];   // only vertices < n are ever marked
            uint32_t e = (uint32_t)a.R[v];
            const uint32_t e1 = (uint32_t)a.R[v + 1];
            if (!VIS && a.depth[v] >= 0) continue;
            a.depth[v] = L;
            found = 1;
            for (; e < e1; e += 8) {
                int32_t u[8];
                uint32_t d[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) u[k] = a.C[entry_or_last(e, k, e1)];
#pragma unroll
                for (int k = 0; k < 8; ++k) d[k] = VIS ? a.vis[u[k] >> 5] >> (u[k] & 31) & 1u : (uint32_t)(a.depth[u[k]] >= 0);
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    if (e + k < e1 && !d[k]) nxt[u[k]] = 1;
                }
            }
        }
        __syncthreads();   // the list is reused by the next span
    }
    if (launch > 0 && blockIdx.x == 0) {
        // the previous level held no vertex: it was the end
        const uint32_t *fprev = a.flags + (size_t)((L & 1) ^ 1) * G;
        uint32_t any = 0;
        for (uint32_t i = threadIdx.x; i < G; i += BLOCK) any |= fprev[i];
        if (!__syncthreads_or((int)any)) {
            if (threadIdx.x == 0) {
                ctl->level = L - 1;
                ctl->push_levels = (uint32_t)(L - 1);
                ctl->dir = DIR_DONE;
            }
            return;
        }
    }
    found = __syncthreads_or(found);
    if (threadIdx.x == 0) a.flags[(size_t)(L & 1) * G + blockIdx.x] = (uint32_t)found;
}

// rows that one thread takes in a turn or two
static bool bm_thin(const Graph &g) { return g.m <= 9ll * g.n; }

static void run_bfs_bitmap(Ctx &c, Graph &g, int32_t src, int32_t *depth, hipStream_t s, Arena &ar)
{
    const int32_t n = g.n;
    const size_t nb = ((size_t)n + 63) / 64 * 64;
    // 32 vertices per thread where 16 would leave more spans than are resident (four groups per CU).
    // Where rows are long a level is bound by how many of the CUs expand them.  On graphs numbered along
    // their edges a frontier is a few spans at any size; on others it is everywhere, and spans of 8,192
    // vertices leave most CUs idle: 2,048 vertices each, or 4,096 where those fill the chip.  Spans of 8,192 /
    // 4,096 / 2,048: random regular graphs of 100,000 x 16, 100,000 x 64, 300,000 x 100 and 1 M x 32 entries 213 /
    // 160 / 147, 632 / 384 / 295, 1,057 / 565 / 468 and 404 / 288 / 283 us; squares with all neighbours within two
    // steps of 100,000 and 1 M vertices 1,205 / 1,320 / 1,564 and 7,310 / 8,530 / 10,990 us; cubes with 26
    // neighbours of 100,000, 300,000 and 1 M vertices (82, 62 and 31 % of the entries inside 8,192 ids) 646 / 732 /
    // 904, 1,287 / 1,466 / 1,585 and 2,815 / 2,756 / 2,508.
    const bool wide = (size_t)n > (size_t)grid_blocks(c, 4) * BM_BLOCK * 16;
    const bool dense = g.cls == GRAPH_MESH && !bm_thin(g);
    const bool near = g.near >= 0.6;
    const int threads = !dense || wide || (near && n >= 32768) ? BM_BLOCK
                        : near || (size_t)n >= 4096ull * c.num_cu ? 256 : 128;
    const size_t span = (size_t)threads * (wide ? 32 : 16);
    const int G = (int)std::min(((size_t)n + span - 1) / span, (size_t)grid_blocks(c, 16));
    const size_t least = 2 * al256(nb) + al256(8ull * G) + al256(sizeof(BfsCtl));
    // a fixed scratch too small for the visited bitmap does without it
    const bool vis = !ar.fixed || least + al256(nb / 8) <= ar.fixed_bytes;
    ar.reserve(least + (vis ? al256(nb / 8) : 0));
    BmArgs a;
    a.R = g.R.as<int32_t>();
    a.C = g.C.as<int32_t>();
    a.n = n;
    a.depth = depth;
    a.mk[0] = ar.take<uint8_t>(nb);
    a.mk[1] = ar.take<uint8_t>(nb);
    a.vis = vis ? ar.take<uint32_t>(nb / 32) : nullptr;
    a.flags = ar.take<uint32_t>(2ull * G);
    a.ctl = ar.take<BfsCtl>(1);
    Fills()
        .add(depth, 0xFFFFFFFFu, (size_t)n)
        .add(a.mk[0], 0u, (2 * al256(nb) + (vis ? al256(nb / 8) : 0)) / 4)   // marks and bitmap (adjacent)
        .run(s);
    // one thread per vertex: only where no vertex has a long row (64 neighbours on either side of 100,000
    // vertices in a ring: 1,562 levels of 33 us in the head, 9 us as launches)
    const bool head = vis && g.cls == GRAPH_MESH && !dense;
    if (head)
        hipLaunchKernelGGL(bfs_bitmap_head, dim3(1), dim3(BM_SOLO_BLOCK), 0, s, a, src);
    else
        hipLaunchKernelGGL(bfs_bitmap_init, dim3(1), dim3(1), 0, s, a, src);
    GFR_LAUNCH_CHECK();
    int32_t i = 0;
    auto launch = [&]() {
        c.ktimer.run("bfs_bitmap_level", s, [&]() {
            const dim3 grid(G), block(threads);
            if (!vis) hipLaunchKernelGGL((bfs_bitmap_level<512, 32, false>), grid, block, 0, s, a, i);
            else if (wide) hipLaunchKernelGGL((bfs_bitmap_level<512, 32, true>), grid, block, 0, s, a, i);
            else if (threads == 512) hipLaunchKernelGGL((bfs_bitmap_level<512, 16, true>), grid, block, 0, s, a, i);
            else if (threads == 256) hipLaunchKernelGGL((bfs_bitmap_level<256, 16, true>), grid, block, 0, s, a, i);
            else hipLaunchKernelGGL((bfs_bitmap_level<128, 16, true>), grid, block, 0, s, a, i);
        });
        ++i;
    };
    const int32_t launched = run_until_done(c, &a.ctl->dir, DIR_DONE,
                                            g.bitmap_launch_hint.load(std::memory_order_relaxed) + 2,
                                            (int64_t)n + 4, s, launch, sizeof(BfsCtl));
    BfsCtl h;
    memcpy(&h, c.pinned, sizeof(BfsCtl));
    c.stats.v["levels"] += h.level;
    c.stats.v["push_levels"] += h.push_levels;
    c.stats.v["pull_levels"] += 0.0;
    c.stats.v["launches"] += launched;
    c.stats.v["solves"] += 1.0;
    g.bitmap_launch_hint.store(h.level + 1 - (int32_t)h.nf, std::memory_order_relaxed);
}

// ------------------------------------------------------------ small graphs
// A traversal of a small graph is all latency: launches, the compaction's
// look-back and the read-back.  Here one work-group does the whole traversal in
// one launch, with the visited bitmap and the list of discovered vertices
// (the levels one after another) in LDS; a level is then two dependent loads
// (row offsets, columns), a few LDS operations and a barrier.  LANES lanes
// share a vertex; rows of more than BS_LONG entries are put aside and walked by
// the whole work-group, so that a hub does not hold a level up.  (2, 4, 8 and 16
// lanes with rows put aside from 32, 128, 256 and 512 entries: 122, 67, 57 and
// 51 us per call on R-MAT with 1,024 vertices and 21 K entries, 133 us with the
// level launches; the kernel takes 24 us of the 51.  All with a wait for the
// stream; 41 us since the kernel itself tells the host that it is done.)
constexpr int BS_BLOCK = 1024;
constexpr int32_t BS_MAX_N = 32768;     // ids fit 16 bits, the list 64 KB
constexpr int32_t BS_LONG = 512;
constexpr int64_t BS_COST = 196608;     // most entries + 16 vertices

struct BsmArgs {
    const int32_t *R;
    const int32_t *C;
    int32_t n;
    int32_t *depth;
    uint32_t *out;       // pinned: levels, entries, edges, discovered
    uint32_t number;     // of this arrival
};

template <int LANES>
__global__ __launch_bounds__(BS_BLOCK) void bfs_small(BsmArgs a, int32_t src)
{
    constexpr int EPL = LANES == 1 ? 8 : 4;   // entries a lane reads together
    __shared__ uint32_t s_vis[BS_MAX_N / 32];
    __shared__ uint16_t s_list[BS_MAX_N];
    __shared__ uint16_t s_hub[BS_COST / BS_LONG];
    __shared__ uint32_t s_cnt, s_nhub, s_edges, s_entries;
    for (int32_t v = threadIdx.x; v < a.n; v += BS_BLOCK) a.depth[v] = v == src ? 0 : -1;
    s_vis[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        s_list[0] = (uint16_t)src;
        s_cnt = 1;
        s_nhub = s_edges = s_entries = 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) s_vis[src >> 5] = 1u << (src & 31);
    __syncthreads();   // (also orders the first stores to depth[] before those of the levels)
    uint32_t edges = 0, entries = 0;
    int32_t L = 0;
    // entries e0, e0 + step, ... below e1 of one row, EPL at a time
    auto expand = [&](int32_t e0, int32_t e1, int32_t step) {
        for (int32_t e = e0; e < e1; e += step * EPL) {
            int32_t u[EPL];
#pragma unroll
            for (int k = 0; k < EPL; ++k) u[k] = a.C[min(e + k * step, e1 - 1)];
#pragma unroll
            for (int k = 0; k < EPL; ++k) {
                const uint32_t bit = 1u << (u[k] & 31);
                if (e + k * step >= e1 || (s_vis[u[k] >> 5] & bit)) continue;
                if (atomicOr(&s_vis[u[k] >> 5], bit) & bit) continue;
                // claimed: one LDS atomic for the lanes that are here
                const uint64_t m = ballot(true);
                const uint32_t below = lanes_below(m);
                uint32_t at = 0;
                if (below == 0) at = atomicAdd(&s_cnt, (uint32_t)__popcll(m));
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + below;
                s_list[at] = (uint16_t)u[k];
                a.depth[u[k]] = L + 1;
            }
        }
    };
    uint32_t lo = 0, hi = 1;
    for (; lo < hi; ++L) {
        for (uint32_t i = lo + threadIdx.x / LANES; i < hi; i += BS_BLOCK / LANES) {
            const int32_t v = s_list[i];
            const int32_t e0 = a.R[v], e1 = a.R[v + 1];
            if (threadIdx.x % LANES == 0 && e1 > e0) {
                edges += (uint32_t)(e1 - e0);
                ++entries;
            }
            if (e1 - e0 > BS_LONG) {
                if (threadIdx.x % LANES == 0) s_hub[atomicAdd(&s_nhub, 1u)] = (uint16_t)v;
            } else {
                expand(e0 + (int32_t)(threadIdx.x % LANES), e1, LANES);
            }
        }
        __syncthreads();
        const uint32_t nhub = s_nhub;
        if (nhub) {   // uniform
            for (uint32_t h = 0; h < nhub; ++h) {
                const int32_t v = s_hub[h];
                expand(a.R[v] + (int32_t)threadIdx.x, a.R[v + 1], BS_BLOCK);
            }
            __syncthreads();
            if (threadIdx.x == 0) s_nhub = 0;
        }
        lo = hi;
        hi = s_cnt;
        __syncthreads();
    }
    if (edges) atomicAdd(&s_edges, edges);
    if (entries) atomicAdd(&s_entries, entries);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // every wave's depths have left it
    __syncthreads();
    if (threadIdx.x == 0) {
        a.out[0] = (uint32_t)L;
        a.out[1] = s_entries;
        a.out[2] = s_edges;
        a.out[3] = s_cnt - 1u;
        arrive(a.out, a.number);
    }
}

// Where one work-group is faster than the chip.  Per call, R-MAT with 4 or 16
// edges drawn per vertex: 8,192 vertices and 57 K entries 103 us (125 by level
// launches), 4,096 and 110 K 97 (118); beyond the line, 16,384 and 116 K 171
// (128), 8,192 and 220 K 166 (120).  With the waits and compactions of today
// 8,192 and 59 K 93 (103), 4,096 and 97 K 85 (89), and the level launches 114
// and 100 beyond the line.  Rows of at most 16 entries (lattices) take
// a thread each, and as many of them as fit the list while they take one turn
// of eight entries: 33^2, 100^2 and 181^2 81, 130 and 248 us (303, 441 and 656
// before).  Rows of two turns reach the line earlier: random regular graphs of 16,384
// vertices with 10 and 16 entries each 143 and 147 us, of 24,576 193 and 196 (131 and
// 139 by level launches), of 32,768 with 8 and 12 entries 165 and 242 (141 and 137).
constexpr int64_t BS_TURNS = 49152;     // most vertices + entries / 8 with rows of two turns
static bool bfs_small_fits(const Ctx &c, const Graph &g)
{
    const Options &o = c.opt;
    const bool fits = g.max_deg <= 8 || (g.max_deg <= 16 && g.n + g.m / 8 <= BS_TURNS) ||
                      g.m + 16ll * g.n <= BS_COST;
    return g.n <= BS_MAX_N && fits && o.bfs_direction != 2 && o.bfs_frontier == 0 && o.advance_mapping == 1 &&
           !o.step_graphs;
}

static void run_bfs_small(Ctx &c, Graph &g, int32_t src, int32_t *depth, hipStream_t s)
{
    const BsmArgs a{g.R.as<int32_t>(), g.C.as<int32_t>(), g.n, depth, c.pinned, ++c.arrivals};
    c.ktimer.run("bfs_small_level", s, [&]() {
        if (g.max_deg <= 16) hipLaunchKernelGGL(bfs_small<1>, dim3(1), dim3(BS_BLOCK), 0, s, a, src);
        else hipLaunchKernelGGL(bfs_small<16>, dim3(1), dim3(BS_BLOCK), 0, s, a, src);
    });
    GFR_LAUNCH_CHECK();
    await_arrival(c, s);
    const volatile uint32_t *h = c.pinned;
    // (queue levels, which scale-free graphs take otherwise, count none from a source without edges)
    const double levels = g.cls == GRAPH_SCALEFREE && h[2] == 0 ? 0.0 : (double)h[0];
    c.stats.v["levels"] += levels;
    c.stats.v["push_levels"] += levels;
    c.stats.v["edges_inspected"] += h[2];
    c.stats.v["push_entries"] += h[1];
    c.stats.v["push_edges"] += h[2];
    c.stats.v["push_new"] += h[3];
    for (const char *k : {"pull_levels", "pull_unvisited", "pull_inspected", "pull_new"}) c.stats.v[k] += 0.0;
    c.stats.v["launches"] += 1.0;
    c.stats.v["solves"] += 1.0;
}

void run_bfs(Ctx &c, Graph &g, int32_t src, int32_t *depth, hipStream_t s)
{
    run_bfs(c, g, src, depth, s, c.arena);
    c.waited = true;   // each path ends with a read-back
}

void run_bfs(Ctx &c, Graph &g, int32_t src, int32_t *depth, hipStream_t s, Arena &ar)
{
    if (bfs_small_fits(c, g)) {
        run_bfs_small(c, g, src, depth, s);
        return;
    }
    const int32_t n = g.n;
    const uint32_t chunk = (uint32_t)c.opt.advance_chunk;
    const uint32_t nwords = (uint32_t)(((int64_t)n + 63) / 64) * 2u;
    const size_t nparts = (size_t)(g.m / chunk) + 2;
    const int G = grid_blocks(c, 8);   // eight work-groups per CU fit at the default chunk
    const CompactGeom cg = compact_geom(nwords, c.num_cu);
    size_t need = 2 * al256(nwords * 4ull) + al256(nwords * 32ull) + 3 * al256(4ull * n) + al256(4 * nparts) +
                  al256(4ull * G) + al256(16ull * cg.blocks) + al256(sizeof(BfsCtl));
    // Mark-byte levels (bfs.frontier 0 auto, 1 queue, 2 mark bytes) on mesh-like graphs; a forced pull
    // direction needs the queue's frontier bitmap.  What decides is the number of levels, which is not
    // known beforehand, and a queue level costs 20 us or more: cubes of 36,000, 300,000 and 3 M vertices
    // with 26 neighbours each (31 to 128 levels) 420 / 680, 1,600 / 1,760 and 5,050 / 7,990 us (marks / queue),
    // squares of 100,000 and 1 M vertices with 24 (106 and 334 levels) 1,205 / 3,620 and 7,310 / 20,300, random regular
    // graphs of 1 M vertices with 10, 16 and 32 entries each (9, 8 and 6 levels) 208 / 262, 225 / 290 and
    // 295 / 285; with 32 entries and 3 M vertices 870 / 425.
    const int fr = c.opt.bfs_frontier;
    if (c.opt.bfs_direction != 2 && (fr == 2 || (fr == 0 && g.cls == GRAPH_MESH))) {
        run_bfs_bitmap(c, g, src, depth, s, ar);
        return;
    }
    ar.reserve(need);
    BfsArgs a;
    memset(&a, 0, sizeof a);   // padding too: the bytes key the captured steps
    a.R = g.R.as<int32_t>();
    a.C = g.C.as<int32_t>();
    a.n = n;
    a.nwords = nwords;
    a.depth = depth;
    a.vis = ar.take<uint32_t>(nwords);
    a.fb = ar.take<uint32_t>(nwords);
    a.mark = ar.take<uint8_t>(32ull * nwords);
    a.q.v = ar.take<int32_t>(n);
    a.q.off = ar.take<uint32_t>(n);
    a.q.row = ar.take<int32_t>(n);
    a.q.part = ar.take<int32_t>(nparts);
    a.likely = g.likely.as<int32_t>();
    a.part_insp = ar.take<uint32_t>(G);
    a.mapping = (uint32_t)c.opt.advance_mapping;
    a.twc_threshold = (uint32_t)c.opt.twc_threshold;
    unsigned long long *status = ar.take<unsigned long long>(2ull * cg.blocks);
    a.ctl = ar.take<BfsCtl>(1);

    const uint32_t bit = 1u << (src & 31);
    fill_first(Fills()
                   .add(depth, 0xFFFFFFFFu, (size_t)n).but((size_t)src, 0u)
                   .add(a.vis, 0u, nwords).but((size_t)src >> 5, bit)
                   .add(a.fb, 0u, nwords).but((size_t)src >> 5, bit)
                   .add(a.mark, 0u, 8ull * nwords)
                   .add(status, 0u, 4ull * cg.blocks),
               BfsFirst{a, src, chunk, (uint32_t)c.opt.bfs_direction, (uint32_t)c.opt.bfs_dedup,
                        (float)c.opt.bfs_alpha, (float)c.opt.bfs_beta, (unsigned long long)g.m},
               s);

    BfsMarks marks{a, (uint32_t)G};
    auto launch = [&]() {
        c.ktimer.run("bfs_level", s, [&]() {
            switch (chunk) {
            case 256: hipLaunchKernelGGL(bfs_level<256>, dim3(G), dim3(GFR_BLOCK), 0, s, a); break;
            case 512: hipLaunchKernelGGL(bfs_level<512>, dim3(G), dim3(GFR_BLOCK), 0, s, a); break;
            case 1024: hipLaunchKernelGGL(bfs_level<1024>, dim3(G), dim3(GFR_BLOCK), 0, s, a); break;
            case 2048: hipLaunchKernelGGL(bfs_level<2048>, dim3(G), dim3(GFR_BLOCK), 0, s, a); break;
            default: hipLaunchKernelGGL(bfs_level<4096>, dim3(G), dim3(GFR_BLOCK), 0, s, a); break;
            }
        });
        c.ktimer.run("bfs_compact", s, [&]() {
            hipLaunchKernelGGL(compact_kernel<BfsMarks>, dim3(cg.blocks), dim3(GFR_BLOCK), 0, s, a.R, n, nwords,
                               cg.wpt, marks, a.q, chunk, status, &a.ctl->parity, &a.ctl->err,
                               c.in_order ? nullptr : &a.ctl->ticket);
        });
    };
    // (no captured steps over fixed scratch: instantiating a graph may allocate)
    StepKey key("bfs");
    key.add(a).add(G).add(cg).add(chunk).add(status).add(c.in_order);
    const int32_t launched = run_until_done(c, &a.ctl->dir, DIR_DONE, g.levels_hint() + 1,
                                            (int64_t)n + 4, s, launch, sizeof(BfsCtl),
                                            ar.fixed ? nullptr : &key);
    BfsCtl h;
    memcpy(&h, c.pinned, sizeof(BfsCtl));
    if (h.err) fail_crowded("bfs");
    c.stats.v["levels"] += h.level;
    c.stats.v["push_levels"] += h.push_levels;
    c.stats.v["pull_levels"] += h.pull_levels;
    c.stats.v["edges_inspected"] += (double)(h.push_edges + h.pull_inspected);
    c.stats.v["push_entries"] += (double)h.push_entries;
    c.stats.v["push_edges"] += (double)h.push_edges;
    c.stats.v["push_new"] += (double)h.push_new;
    c.stats.v["pull_unvisited"] += (double)h.pull_unvisited;
    c.stats.v["pull_inspected"] += (double)h.pull_inspected;
    c.stats.v["pull_new"] += (double)h.pull_new;
    c.stats.v["launches"] += launched;
    c.stats.v["solves"] += 1.0;
    g.bfs_levels_hint.store(h.level, std::memory_order_relaxed);
}

}  // namespace gfr
