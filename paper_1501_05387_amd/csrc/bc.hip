// bc.hip -- betweenness centrality from a set of sources, Brandes'
// two-pass formulation as the paper maps it (Sec. 5.3):
//   forward   an advance identical to BFS discovers level L+1 from level L,
//             pushing from the level's lists or, when the level is large,
//             pulling: every unvisited vertex scans its own list for a vertex
//             of level L (the direction choice of Sec. 4.5, which the paper
//             names as the missing piece of its BC); then a compute step
//             gathers sigma(v) = sum of sigma(u) over the neighbours u one
//             level up (shortest-path counts, FP64);
//   backward  walks the levels in reverse and gathers
//             delta(v) = sigma(v) * sum over neighbours w one level down of
//                        (1 + delta(w)) / sigma(w),
//             stored in FP32; bc(v) accumulates delta(v) over sources.
// Both gathers are pull-style: no floating-point atomics, fixed order per
// list (see gather.h).  Depths are kept as one byte per vertex, depth mod
// 128 (0xFF = unvisited): the neighbours a gather inspects are within one
// level of the gathering vertex (or not yet discovered), so the byte
// identifies the level exactly, and the array is a quarter of an int32 one,
// which keeps the random probes of the gathers in cache.  Every level is kept as a contiguous slice of one BFS
// order array so the backward pass can revisit it.
#include <vector>

#include "compact.h"
#include "engine.h"
#include "gather.h"

namespace gfr {

constexpr uint8_t BC_UNSEEN = 0xFF;   // never a level code

__host__ __device__ __forceinline__ uint8_t level_code(int32_t L) { return (uint8_t)(L & 127); }
static_assert(BC_UNSEEN > 127, "unvisited must differ from every level code");

struct BcArgs {
    const int32_t *R;
    const int32_t *C;
    uint8_t *dc;     // depth code per vertex
    uint32_t *vis;
};

// One level of the forward pass: where its vertices lie in the BFS order.
struct BcLevel {
    uint32_t mf, nf;         // edges, entries (0, 0: not reached)
    uint32_t start, pbase;   // first entry and first chunk index
};

// The forward pass runs from device memory alone: the host queues levels ahead
// (each launch knows its level) and waits once per source, for their number.
// Waiting for every level's size took about 25 us a level.
struct BcCtl {
    uint32_t done;           // first word: read back by the host
    uint32_t levels;         // levels found
    uint32_t pull;           // the next discovery pulls
    uint32_t parity, err, ticket;    // of the compaction
    uint32_t force;          // 0 auto, 1 push, 2 pull
    uint32_t push_levels, pull_levels;
    double mu, prev_nf;      // edges of unvisited vertices; size of the level before
    double alpha, beta;
};

// the direction of the discovery from a level of nf vertices and mf edges
__device__ __forceinline__ uint32_t bc_direction(const BcCtl *ctl, uint32_t nf, uint32_t mf, int32_t n)
{
    if (ctl->force) return ctl->force == 2;
    if (!ctl->pull) return (double)mf > ctl->mu / ctl->alpha && (double)nf > ctl->prev_nf;
    return !((double)nf < (double)n / ctl->beta && (double)nf < ctl->prev_nf);
}

// push advance of one level (load-balanced edge chunks): an unvisited
// neighbour gets its depth code and a mark byte (plain stores; duplicates write
// the same values and collapse in the compaction)
template <int CH>
__device__ __forceinline__ void bc_push_discover(const BcArgs &a, const FrontierQ &qin, uint32_t nf, uint32_t mf,
                                                 int32_t L, uint8_t *mark)
{
    __shared__ uint32_t s_off[CH + 1];
    __shared__ int32_t s_row[CH + 1];
    const uint32_t nchunks = (mf + CH - 1) / CH;
    for (uint32_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const uint32_t e0 = c * CH;
        const uint32_t e1 = min(e0 + (uint32_t)CH, mf);
        const int s = qin.part[c];
        const int t = (c + 1 < nchunks) ? qin.part[c + 1] : (int)nf - 1;
        const int cnt = t - s + 1;
        __syncthreads();
        for (int i = threadIdx.x; i < cnt; i += GFR_BLOCK) {
            s_off[i] = qin.off[s + i];
            s_row[i] = qin.row[s + i];
        }
        __syncthreads();
        for (uint32_t k = 0; k < (uint32_t)CH; k += GFR_BLOCK) {
            const uint32_t e = e0 + k + threadIdx.x;
            if (e < e1) {
                const int i = upper_index(s_off, 0, cnt - 1, e);
                const int32_t v = a.C[s_row[i] + (int32_t)(e - s_off[i])];
                if (!((a.vis[v >> 5] >> (v & 31)) & 1u) && !mark[v]) {
                    a.dc[v] = level_code(L + 1);
                    mark[v] = 1;
                }
            }
        }
    }
}

// pull discovery of level L+1: every unvisited vertex (lane = vertex) scans
// its list four neighbours at a time until one is in the level-L bitmap
__device__ __forceinline__ void bc_pull_discover(const BcArgs &a, int32_t n, const uint32_t *fb, int32_t L,
                                                 uint8_t *mark)
{
    const uint32_t waves = gridDim.x * GFR_WAVES;
    const int lane = lane_id();
    for (uint32_t grp = blockIdx.x * GFR_WAVES + threadIdx.x / 64; grp * 64u < (uint32_t)n; grp += waves) {
        const int32_t v = (int32_t)(grp * 64u) + lane;
        const uint32_t visw = a.vis[grp * 2u + (uint32_t)(lane >> 5)];
        bool found = false;
        if (v < n && !(visw & (1u << (v & 31)))) {
            uint32_t e = (uint32_t)a.R[v];
            const uint32_t re = (uint32_t)a.R[v + 1];
            while (e < re) {
                const uint32_t k = min(4u, re - e);
                int32_t u[4];
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) u[j] = a.C[j < k ? e + j : e];
                uint32_t hit = 0;
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) hit |= (j < k) ? (fb[u[j] >> 5] >> (u[j] & 31)) & 1u : 0u;
                if (hit) {
                    found = true;
                    break;
                }
                e += 4;
            }
        }
        if (found) {
            a.dc[v] = level_code(L + 1);
            mark[v] = 1;
        }
    }
}

// discovery of level L + 1
template <int CH>
__global__ __launch_bounds__(GFR_BLOCK) void bc_discover(BcArgs a, int32_t n, FrontierQ order, const BcLevel *lv,
                                                         const BcCtl *ctl, const uint32_t *fb, int32_t L,
                                                         uint8_t *mark)
{
    if (ctl->done) return;
    if (ctl->pull) {
        bc_pull_discover(a, n, fb, L, mark);
    } else {
        const BcLevel l = lv[L];
        bc_push_discover<CH>(a, QueueAt{&lv[L].start}(order), l.nf, l.mf, L, mark);
    }
}

// compaction of level L + 1 into its slice of the BFS order (vertex order);
// also writes the level's bitmap for a following pull discovery
struct BcMarks {
    uint8_t *mark;
    uint32_t *vis;
    uint32_t *fb;
    BcLevel *lv;
    BcCtl *ctl;
    int32_t L, n;
    __device__ bool skip() const { return ctl->done != 0; }
    __device__ BcLevel next() const
    {
        const BcLevel l = lv[L];
        return BcLevel{0u, 0u, l.start + l.nf, l.pbase + (l.mf + GATHER_CH - 1) / GATHER_CH + 1u};
    }
    __device__ FrontierQ place(const FrontierQ &q) const
    {
        const BcLevel x = next();
        return FrontierQ{q.v + x.start, q.off + x.start, q.row + x.start, q.part + x.pbase};
    }
    __device__ uint32_t mask(uint32_t w) const
    {
        const uint32_t m = marks_to_mask(mark + 32ull * w);
        if (m) {
            clear_marks(mark + 32ull * w);
            vis[w] |= m;
        }
        fb[w] = m;
        return m;
    }
    __device__ void partial(uint32_t) {}
    __device__ void control(uint32_t nf, uint32_t mf) const
    {
        if (threadIdx.x != 0) return;
        ctl->parity ^= 1u;
        if (ctl->pull) ctl->pull_levels += 1u;
        else ctl->push_levels += 1u;
        if (nf == 0) {
            ctl->done = 1u;
            return;
        }
        BcLevel x = next();
        x.nf = nf;
        x.mf = mf;
        lv[L + 1] = x;
        ctl->levels += 1u;
        ctl->mu -= (double)mf;
        ctl->prev_nf = (double)lv[L].nf;
        ctl->pull = bc_direction(ctl, nf, mf, n);
    }
};

// (lv[] is zero but for what the forward pass writes)
__global__ void bc_source_init(BcArgs a, int32_t src, int32_t n, FrontierQ q0, double *sigma, BcLevel *lv, BcCtl *ctl,
                               uint32_t *fb, uint32_t force, double alpha, double beta)
{
    const int32_t rs = a.R[src], deg = a.R[src + 1] - rs;
    if (threadIdx.x == 0) {
        a.dc[src] = level_code(0);
        a.vis[src >> 5] |= 1u << (src & 31);
        fb[src >> 5] |= 1u << (src & 31);
        sigma[src] = 1.0;
        q0.v[0] = src;
        q0.off[0] = 0;
        q0.row[0] = rs;
        lv[0] = BcLevel{(uint32_t)deg, 1u, 0u, 0u};
        ctl->done = deg == 0;
        ctl->levels = 1;
        ctl->pull = 0;
        ctl->force = force;
        ctl->alpha = alpha;
        ctl->beta = beta;
        ctl->mu = (double)a.R[n] - (double)deg;
        ctl->prev_nf = 0.0;
        ctl->pull = bc_direction(ctl, 1u, (uint32_t)deg, n);
    }
    for (uint32_t c = threadIdx.x; (uint64_t)c * GATHER_CH < (uint64_t)deg; c += blockDim.x) q0.part[c] = 0;
}

struct SigmaOp {
    const uint8_t *dc;
    const double *sigma;
    uint8_t code;   // level of the predecessors
    __device__ double operator()(int32_t u) const { return dc[u] == code ? sigma[u] : 0.0; }
};

struct SigmaFin {
    double *sigma;
    __device__ void operator()(int32_t v, double s) const { sigma[v] = s; }
};

struct DeltaOp {
    const uint8_t *dc;
    const double *coef;
    uint8_t code;   // level of the successors
    __device__ double operator()(int32_t w) const { return dc[w] == code ? coef[w] : 0.0; }
};

struct DeltaFin {
    const double *sigma;
    double *coef;
    double *bc;
    __device__ void operator()(int32_t v, double s) const
    {
        const float dl = (float)(sigma[v] * s);
        coef[v] = (1.0 + (double)dl) / sigma[v];
        bc[v] += (double)dl;
    }
};

__global__ void bc_leaf_coef(FrontierQ q, const BcLevel *l, const double *sigma, double *coef)
{
    const uint32_t nf = l->nf;
    q = QueueAt{&l->start}(q);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nf; i += gridDim.x * blockDim.x) {
        const int32_t v = q.v[i];
        coef[v] = 1.0 / sigma[v];
    }
}

__global__ void bc_to_f32(const double *acc, float *out, int32_t n)
{
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x)
        out[v] = (float)acc[v];
}

void run_bc(Ctx &c, Graph &g, const int32_t *sources, int32_t k, float *bc, hipStream_t s)
{
    const int32_t n = g.n;
    const uint32_t nwords = (uint32_t)(((int64_t)n + 63) / 64) * 2u;
    const size_t nparts = (size_t)(g.m / GATHER_CH) + 2ull * n + 4;
    const size_t nch = (size_t)(g.m / GATHER_CH) + 2;
    const size_t nlev = (size_t)n + 2;
    c.arena.reserve(al256(4ull * n) + al256(4ull * nwords) + al256(32ull * nwords) + 3 * al256(8ull * n) + 3 * al256(4ull * n) +
                    al256(4 * nparts) + 2 * al256(8 * nch) + al256(sizeof(BcLevel) * nlev) +
                    al256(16ull * (uint64_t)compact_geom(nwords, c.num_cu).blocks) + al256(256) +
                    al256(4ull * nwords));
    BcArgs a;
    a.R = g.R.as<int32_t>();
    a.C = g.C.as<int32_t>();
    a.dc = c.arena.take<uint8_t>(4ull * ((n + 3) / 4));
    a.vis = c.arena.take<uint32_t>(nwords);
    double *sigma = c.arena.take<double>(n);
    double *coef = c.arena.take<double>(n);
    double *acc = c.arena.take<double>(n);
    int32_t *order = c.arena.take<int32_t>(n);
    uint32_t *off = c.arena.take<uint32_t>(n);
    int32_t *row = c.arena.take<int32_t>(n);
    int32_t *part = c.arena.take<int32_t>(nparts);
    GatherScratch gs{c.arena.take<double>(nch), c.arena.take<double>(nch)};
    BcLevel *lv = c.arena.take<BcLevel>(nlev);
    const int G = grid_blocks(c, 4);
    const CompactGeom cg = compact_geom(nwords, c.num_cu);
    uint8_t *mark = c.arena.take<uint8_t>(32ull * nwords);
    unsigned long long *status = c.arena.take<unsigned long long>(2ull * cg.blocks);
    BcCtl *ctl = c.arena.take<BcCtl>(1);
    uint32_t *fb = c.arena.take<uint32_t>(nwords);
    Fills()
        .add(mark, 0u, 8ull * nwords)
        .add(status, 0u, 4ull * cg.blocks)
        .add(ctl, 0u, sizeof(BcCtl) / 4)
        .add(lv, 0u, nlev * sizeof(BcLevel) / 4)
        .add(acc, 0u, 2ull * n)
        .run(s);
    const FrontierQ q{order, off, row, part};
    const uint32_t *zero = c.zero_word.as<uint32_t>();
    const dim3 grid(G), block(GFR_BLOCK);
    double levels_total = 0;
    BcCtl h{};
    uint32_t used = 1;   // levels of the source before
    for (int32_t si = 0; si < k; ++si) {
        const int32_t src = sources[si];
        Fills()
            .add(a.dc, 0xFFFFFFFFu, (n + 3) / 4)   // BC_UNSEEN
            .add(a.vis, 0u, nwords)
            .add(fb, 0u, nwords)
            .add(lv, 0u, used * sizeof(BcLevel) / 4)
            .run(s);
        hipLaunchKernelGGL(bc_source_init, dim3(1), block, 0, s, a, src, n, q, sigma, lv, ctl, fb,
                           (uint32_t)c.opt.bc_direction, c.opt.bc_alpha, c.opt.bc_beta);
        GFR_LAUNCH_CHECK();
        // forward: launch i discovers level i + 1 and counts its paths
        int32_t L = 0;
        auto launch = [&]() {
            if (L > n) return;   // (there are at most n levels)
            hipLaunchKernelGGL(bc_discover<GATHER_CH>, grid, block, 0, s, a, n, q, lv, ctl, fb, L, mark);
            hipLaunchKernelGGL(compact_kernel<BcMarks>, dim3(cg.blocks), block, 0, s, a.R, n, nwords, cg.wpt,
                               BcMarks{mark, a.vis, fb, lv, ctl, L, n}, q, GATHER_CH, status, &ctl->parity, &ctl->err,
                               c.in_order ? nullptr : &ctl->ticket);
            const BcLevel *x = lv + L + 1;
            const QueueAt at{&x->start};
            hipLaunchKernelGGL((gather_chunks<GATHER_CH, SigmaOp, SigmaFin>), grid, block, 0, s, q, &x->nf, &x->mf,
                               a.C, SigmaOp{a.dc, sigma, level_code(L)}, SigmaFin{sigma}, gs, zero, at);
            hipLaunchKernelGGL((gather_fixup<GATHER_CH, SigmaFin>), grid, block, 0, s, q, &x->nf, &x->mf,
                               SigmaFin{sigma}, gs, zero, at);
            ++L;
        };
        const int32_t hint = g.bc_levels_hint.load(std::memory_order_relaxed);
        run_until_done(c, &ctl->done, 1u, hint + hint / 32, (int64_t)n + 8, s, launch, sizeof(BcCtl));
        memcpy(&h, c.pinned, sizeof h);
        if (h.err) fail_crowded("bc");
        g.bc_levels_hint.store((int32_t)h.levels, std::memory_order_relaxed);
        used = h.levels + 1;
        levels_total += (double)h.levels;
        // backward: the deepest level has no successors
        const int32_t Lmax = (int32_t)h.levels - 1;
        if (Lmax >= 1) hipLaunchKernelGGL(bc_leaf_coef, grid, block, 0, s, q, lv + Lmax, sigma, coef);
        for (int32_t l = Lmax - 1; l >= 1; --l) {
            const QueueAt at{&lv[l].start};
            hipLaunchKernelGGL((gather_chunks<GATHER_CH, DeltaOp, DeltaFin>), grid, block, 0, s, q, &lv[l].nf,
                               &lv[l].mf, a.C, DeltaOp{a.dc, coef, level_code(l + 1)}, DeltaFin{sigma, coef, acc}, gs,
                               zero, at);
            hipLaunchKernelGGL((gather_fixup<GATHER_CH, DeltaFin>), grid, block, 0, s, q, &lv[l].nf, &lv[l].mf,
                               DeltaFin{sigma, coef, acc}, gs, zero, at);
        }
        GFR_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(bc_to_f32, dim3(G), dim3(GFR_BLOCK), 0, s, acc, bc, n);
    GFR_LAUNCH_CHECK();
    c.stats.v["levels"] = levels_total;
    c.stats.v["push_levels"] = (double)h.push_levels;   // summed over the sources
    c.stats.v["pull_levels"] = (double)h.pull_levels;
}

}  // namespace gfr
