// cc.hip -- connected components by hooking and pointer jumping (Sec. 5.4).
//
// label[] is a forest of parent pointers with label[v] <= v.  Hooking an edge
// climbs from both ends to a common ancestor; where the ends meet in two
// different roots, the larger is hooked under the smaller by a compare-and-swap
// on the root itself.  Pointer jumping flattens every tree to a star.  Because
// a root is only ever hooked under a smaller vertex of its component, the root
// that survives is the component's smallest id, the label convention of this
// library, whatever the order of the hooks.
//
// What a round costs is its pass over the edges, so most edges are never
// looked at (a filter of the edge frontier by its endpoints' labels, Sec. 5.4,
// before the edges are read): a vertex first hooks along its first neighbour
// only (no atomics: it is the pointer's initial value), then along its second,
// and these two leave nearly all vertices of the largest component in one
// star.  Its label is read off a sample, and the sweep that hooks over whole
// lists skips every vertex that carries it: an edge between such a vertex and
// another component is hooked from the other side (graphs are stored
// symmetrically).  The sample only decides what is skipped, never the result.
// Hooking few neighbours first and leaving out the sampled component is the
// neighbour sampling of Sutton, Ben-Nun and Barak (Afforest, IPDPS 2018); climbs
// that write back the ancestors they reach are known from Jaiganesh and
// Burtscher (ECL-CC, HPDC 2018).
//
// Two sweeps over all edges, hooking with atomicMin, took 3.0 ms each on the
// 3001^2 lattice (35 M entries) and the call 6.6 ms.  This
// form takes 0.42 ms there, of which the first flattening is 0.17 ms.
#include "engine.h"
#include "gather.h"

namespace gfr {

// Join the trees of a and b.  Every turn replaces the larger end by its parent,
// which is smaller, so the loop ends; a parent that is out of date is an
// ancestor all the same, and only the compare-and-swap decides that it is a root.
__device__ __forceinline__ void hook(int32_t *label, int32_t a, int32_t b)
{
    while (a != b) {
        const int32_t hi = a > b ? a : b, lo = a > b ? b : a;
        int32_t p = label[hi];   // from before another group's hook at worst
        if (p == hi) {
            p = atomicCAS(label + hi, hi, lo);
            if (p == hi) return;
        }
        a = p;
        b = lo;
    }
}

// first neighbours: a vertex starts below its first neighbour if that is smaller
__global__ __launch_bounds__(GFR_BLOCK) void cc_init(const int32_t *R, const int32_t *C, int32_t *label, int32_t n)
{
    for (int64_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const int32_t e = R[v];
        label[v] = e < R[v + 1] ? min((int32_t)v, C[e]) : (int32_t)v;
    }
}

// second neighbours
__global__ __launch_bounds__(GFR_BLOCK) void cc_hook_second(const int32_t *R, const int32_t *C, int32_t *label,
                                                            int32_t v0, int32_t n)
{
    for (int64_t v = (int64_t)v0 + blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const int32_t e = R[v] + 1;
        if (e < R[v + 1]) hook(label, label[v], label[C[e]]);
    }
}

// Flatten the trees of the first n vertices.  A climb writes back each ancestor
// it reaches, which shortens the climbs of its neighbours in flight (a lattice
// column is a chain of as many links as the lattice has rows).  What the other
// XCDs write back is not asked for: an old value is an ancestor all the same,
// and loads at device scope made the first flattening of the 3001^2 lattice
// 306 us against 166.  Two, four and eight climbs per thread took 690, 1,328
// and 2,028 us: the climbs then start far above the part that is already flat.
// With `part`, each work-group also counts its roots.
__global__ __launch_bounds__(GFR_BLOCK) void cc_jump(int32_t *label, int32_t n, uint32_t *part)
{
    uint32_t roots = 0;
    for (int64_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        int32_t r = label[v];
        if (r == (int32_t)v) {
            ++roots;
            continue;
        }
        int32_t p = label[r];
        while (p != r) {
            __hip_atomic_store(label + v, p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            r = p;
            p = __hip_atomic_load(label + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    if (!part) return;
    __shared__ uint32_t s[GFR_WAVES];
    roots = wave_sum_u32(roots);
    if (lane_id() == 0) s[threadIdx.x / 64] = roots;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int i = 0; i < GFR_WAVES; ++i) t += s[i];
        part[blockIdx.x] = t;
    }
}

// *most = the label that most of GFR_BLOCK vertices spread over the ids carry (one work-group)
__global__ __launch_bounds__(GFR_BLOCK) void cc_sample(const int32_t *label, int32_t n, int32_t *most)
{
    __shared__ int32_t s_l[GFR_BLOCK];
    __shared__ uint32_t s_best;
    const int32_t mine = label[(int64_t)n * threadIdx.x / GFR_BLOCK];
    s_l[threadIdx.x] = mine;
    if (threadIdx.x == 0) s_best = 0;
    __syncthreads();
    uint32_t same = 0;
    for (int i = 0; i < GFR_BLOCK; ++i) same += s_l[i] == mine;
    const uint32_t key = (same << 8) | threadIdx.x;   // same <= 256
    atomicMax(&s_best, key);
    __syncthreads();
    if (s_best == key) *most = mine;
}

// Hook along every edge of the vertices outside the sampled component, equal
// edge chunks per work-group.  q: the whole vertex set, whose edge offsets are
// the row offsets themselves, so edge e of the chunk is entry e of C.
__global__ __launch_bounds__(GFR_BLOCK) void cc_hook_rest(FrontierQ q, uint32_t nf, uint32_t mf, const int32_t *C,
                                                          int32_t *label, const int32_t *most)
{
    constexpr uint32_t CH = GATHER_CH;
    __shared__ uint32_t s_off[CH + 1];
    __shared__ int32_t s_v[CH + 1];   // -1: skipped
    const int32_t skip = *most;
    const uint32_t nchunks = (mf + CH - 1) / CH;
    for (uint32_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const uint32_t e0 = c * CH, e1 = min(e0 + CH, mf);
        const int s = q.part[c];
        const int t = (c + 1 < nchunks) ? q.part[c + 1] : (int)nf - 1;
        const int cnt = t - s + 1;
        int any = 0;
        for (int i = threadIdx.x; i < cnt; i += GFR_BLOCK) {
            const int32_t v = q.v[s + i];
            const bool take = label[v] != skip;
            s_off[i] = q.off[s + i];
            s_v[i] = take ? v : -1;
            any |= take;
        }
        if (__syncthreads_or(any)) {
            for (uint32_t e = e0 + threadIdx.x; e < e1; e += GFR_BLOCK) {
                const int32_t v = s_v[upper_index(s_off, 0, cnt - 1, e)];
                if (v >= 0) hook(label, label[v], label[C[e]]);
            }
        }
        __syncthreads();   // the next chunk rewrites the LDS arrays
    }
}

__global__ __launch_bounds__(GFR_BLOCK) void cc_sum(const uint32_t *part, uint32_t nparts, uint32_t *out)
{
    uint32_t r = 0;
    for (uint32_t i = threadIdx.x; i < nparts; i += GFR_BLOCK) r += part[i];
    __shared__ uint32_t s[GFR_WAVES];
    r = wave_sum_u32(r);
    if (lane_id() == 0) s[threadIdx.x / 64] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int i = 0; i < GFR_WAVES; ++i) t += s[i];
        *out = t;
    }
}

void run_cc(Ctx &c, Graph &g, int32_t *label, int32_t *ncomp, hipStream_t s)
{
    const int32_t n = g.n;
    const int G = grid_blocks(c, 8);
    c.arena.reserve(al256(4ull * G) + al256(8));
    uint32_t *rpart = c.arena.take<uint32_t>(G);
    uint32_t *word = c.arena.take<uint32_t>(2);   // [0] sampled label, [1] roots
    const int32_t *R = g.R.as<int32_t>(), *C = g.C.as<int32_t>();
    const dim3 grid(G), block(GFR_BLOCK);
    uint32_t *none = nullptr;
    hipLaunchKernelGGL(cc_init, grid, block, 0, s, R, C, label, n);
    if (g.full_nf) {
        hipLaunchKernelGGL(cc_jump, grid, block, 0, s, label, n, none);
        // the first part joins what it can; flattening it keeps the climbs of the rest short
        hipLaunchKernelGGL(cc_hook_second, grid, block, 0, s, R, C, label, 0, n / 64);
        hipLaunchKernelGGL(cc_jump, grid, block, 0, s, label, n / 64, none);
        hipLaunchKernelGGL(cc_hook_second, grid, block, 0, s, R, C, label, n / 64, n);
        hipLaunchKernelGGL(cc_jump, grid, block, 0, s, label, n, none);
        hipLaunchKernelGGL(cc_sample, dim3(1), block, 0, s, label, n, (int32_t *)word);
        hipLaunchKernelGGL(cc_hook_rest, grid, block, 0, s, g.full, (uint32_t)g.full_nf, (uint32_t)g.m, C, label,
                           (const int32_t *)word);
    }
    hipLaunchKernelGGL(cc_jump, grid, block, 0, s, label, n, rpart);
    hipLaunchKernelGGL(cc_sum, dim3(1), block, 0, s, rpart, (uint32_t)G, word + 1);
    GFR_LAUNCH_CHECK();
    read_back(c, word + 1, 4, s);
    c.waited = true;
    *ncomp = (int32_t)c.pinned[0];
    c.stats.v["rounds"] = 3;   // first neighbours, second neighbours, the rest
}

}  // namespace gfr
