// ranked.hip -- columns renumbered by degree for the whole-graph gathers of
// hotgather.h: a counting sort of the vertices with edges into 256 classes of
// degree (eight per power of two, highest first), then one pass over the
// columns.  The order inside a class is the order in which work-groups claim
// their places; it decides where a value is stored, never what is summed or in
// which order.
#include "hotgather.h"

namespace gfr {

constexpr int RANK_GROUPS = 1024;

// 255 - (eight classes per power of two), so that high degrees come first; d >= 1
__device__ __forceinline__ uint32_t degree_class(uint32_t d)
{
    const uint32_t l = 31u - (uint32_t)__clz(d);
    return 255u - (l * 8u + ((l >= 3u ? d >> (l - 3u) : d << (3u - l)) & 7u));
}

struct RankArgs {
    const uint32_t *off;    // [nf] of the whole-graph queue
    const int32_t *v;
    uint32_t nf, mf;
    uint32_t *cursor;       // [256] class sizes, then next free places
    int32_t *pos;           // [n] place of each vertex with edges; nf of the others
    int32_t *epos;          // [nf] the same by entry
};

// pass 0: class sizes; pass 1: places (each work-group claims a run per class)
template <int PASS>
__global__ __launch_bounds__(256) void rank_pass(RankArgs a)
{
    __shared__ uint32_t s_n[256], s_base[256];
    const uint32_t per = (a.nf + gridDim.x - 1) / gridDim.x;
    const uint32_t lo = min(a.nf, blockIdx.x * per), hi = min(a.nf, lo + per);
    auto degree = [&](uint32_t i) { return (i + 1 < a.nf ? a.off[i + 1] : a.mf) - a.off[i]; };
    s_n[threadIdx.x] = 0;
    __syncthreads();
    for (uint32_t i = lo + threadIdx.x; i < hi; i += 256) atomicAdd(&s_n[degree_class(degree(i))], 1u);
    __syncthreads();
    const uint32_t mine = s_n[threadIdx.x];
    if (PASS == 0) {
        if (mine) atomicAdd(a.cursor + threadIdx.x, mine);
        return;
    }
    s_base[threadIdx.x] = mine ? atomicAdd(a.cursor + threadIdx.x, mine) : 0u;
    s_n[threadIdx.x] = 0;
    __syncthreads();
    for (uint32_t i0 = lo; i0 < hi; i0 += 256) {   // ascending ids stay together inside a class
        const uint32_t i = i0 + threadIdx.x;
        if (i < hi) {
            const uint32_t k = degree_class(degree(i));
            const int32_t p = (int32_t)(s_base[k] + atomicAdd(&s_n[k], 1u));
            a.pos[a.v[i]] = p;
            a.epos[i] = p;
        }
        __syncthreads();
    }
}

// class sizes -> first places
__global__ __launch_bounds__(256) void rank_scan(uint32_t *cursor)
{
    __shared__ uint32_t s_w[4];
    const uint32_t x = cursor[threadIdx.x], incl = wave_incl_scan(x);
    if (lane_id() == 63) s_w[threadIdx.x / 64] = incl;
    __syncthreads();
    uint32_t before = 0;
    for (int w = 0; w < (int)(threadIdx.x / 64); ++w) before += s_w[w];
    cursor[threadIdx.x] = before + incl - x;
}

__global__ __launch_bounds__(256) void rank_columns(const int32_t *C, const int32_t *pos, uint32_t m, uint32_t padded,
                                                    int32_t *out)
{
    for (uint64_t e = ((uint64_t)blockIdx.x * 256 + threadIdx.x) * 4; e < padded; e += (uint64_t)gridDim.x * 1024) {
        int4 x = make_int4(0, 0, 0, 0);
        if (e + 4 <= m) {
            const int4 u = *(const int4 *)(C + e);
            x = make_int4(pos[u.x], pos[u.y], pos[u.z], pos[u.w]);
        } else {
            if (e < m) x.x = pos[C[e]];
            if (e + 1 < m) x.y = pos[C[e + 1]];
            if (e + 2 < m) x.z = pos[C[e + 2]];
        }
        *(int4 *)(out + e) = x;
    }
}

__global__ __launch_bounds__(256) void rank_starts(const uint32_t *off, uint32_t nf, uint32_t *starts)
{
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < nf; i += gridDim.x * 256)
        atomicOr(starts + (off[i] >> 5), 1u << (off[i] & 31u));
}

__global__ __launch_bounds__(256) void rank_entries(FrontierQ full, uint32_t nf, uint32_t mf, uint32_t nch,
                                                    int32_t *entry)
{
    constexpr uint32_t PER = GATHER_CH / HG_CH;   // the queue's own chunk index narrows the search
    const uint32_t nparts = (mf + GATHER_CH - 1) / GATHER_CH;
    for (uint32_t c = blockIdx.x * 256 + threadIdx.x; c < nch; c += gridDim.x * 256) {
        const uint32_t p = c / PER;
        const int lo = full.part[p], hi = p + 1 < nparts ? full.part[p + 1] : (int)nf - 1;
        entry[c] = upper_index(full.off, lo, hi, c * HG_CH);
    }
}

const RankedCols *ranked_cols(Ctx &c, Graph &g, hipStream_t s)
{
    RankedCols &r = g.ranked;
    const auto make = [&]() {
        const uint32_t m = (uint32_t)g.m;
        const uint32_t nch = (m + HG_CH - 1) / HG_CH;
        const size_t padded = (size_t)nch * HG_CH;
        const uint32_t nf = (uint32_t)g.full_nf;
        const size_t b_c = al256(4 * padded), b_p = al256(4ull * nf), b_s = al256(padded / 8 + HG_CH / 8),
                     b_e = al256(4ull * (nch + 1));
        c.arena.reserve(al256(4ull * g.n));
        int32_t *pos = c.arena.take<int32_t>(g.n);   // by vertex: only the columns need it
        r.mem.alloc(b_c + b_p + b_s + b_e + 1024);
        char *base = (char *)r.mem.p;
        r.C = (int32_t *)base;
        r.pos = (int32_t *)(base + b_c);
        r.starts = (uint32_t *)(base + b_c + b_p);
        r.entry = (int32_t *)(base + b_c + b_p + b_s);
        uint32_t *cursor = (uint32_t *)(base + b_c + b_p + b_s + b_e);
        r.nch = nch;
        const dim3 grid(grid_blocks(c, 8)), block(256);
        fill_u32(cursor, 0u, 256, s);
        fill_u32(r.starts, 0u, b_s / 4, s);
        // In a symmetric graph every target has edges.  The load does not ask for symmetry unless it is told to
        // validate, so a target without edges gets the table's last place, which holds 0.
        fill_u32(pos, nf, (size_t)g.n, s);
        const RankArgs a{g.full.off, g.full.v, nf, m, cursor, pos, r.pos};
        hipLaunchKernelGGL(rank_pass<0>, dim3(RANK_GROUPS), block, 0, s, a);
        hipLaunchKernelGGL(rank_scan, dim3(1), block, 0, s, cursor);
        hipLaunchKernelGGL(rank_pass<1>, dim3(RANK_GROUPS), block, 0, s, a);
        hipLaunchKernelGGL(rank_columns, grid, block, 0, s, g.C.as<int32_t>(), pos, m, (uint32_t)padded, r.C);
        hipLaunchKernelGGL(rank_starts, grid, block, 0, s, g.full.off, nf, r.starts);
        hipLaunchKernelGGL(rank_entries, grid, block, 0, s, g.full, nf, m, nch, r.entry);
        GFR_LAUNCH_CHECK();
        GFR_HIP(hipStreamSynchronize(s));   // later calls may come on other streams
        g.bytes += r.mem.bytes;
    };
    const bool made = r.have.get(make, [&]() {
        (void)hipGetLastError();
        r.mem.release();
    });
    return made ? &r : nullptr;
}

bool give_back_spares(Ctx &c)
{
    bool any = false;
    for (auto &kv : c.graphs) {
        Graph &g = *kv.second;
        if (g.ranked.have.state != Spare::MADE) continue;
        g.bytes -= g.ranked.mem.bytes;
        g.ranked.mem.release();
        g.ranked.have.state = Spare::NO_ROOM;
        any = true;
    }
    if (any) (void)hipGetLastError();   // of the allocation that failed: the call is made again
    return any;
}

HotGraph hot_graph(const Graph &g, const RankedCols &r)
{
    return HotGraph{r.C, r.starts, r.entry, g.full.off, (uint32_t)g.full_nf, (uint32_t)g.m, r.nch};
}

}  // namespace gfr
