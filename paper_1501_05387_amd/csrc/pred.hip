// pred.hip -- predecessor arrays read off finished distances: a BFS tree
// (Sec. 5.1) or a shortest-path tree (Sec. 5.2).  pred[src] = src, -1 where
// unreached, otherwise the first neighbour u in v's row that is one step
// closer to the source (depth[u] = depth[v] - 1, or dist[u] + w = dist[v]).
// Taking the first such neighbour in row order makes the result unique (the
// smallest id when rows are sorted) instead of whichever discoverer won a
// race during the traversal.
//
// A row is scanned only as far as its first hit, so what bounds the pass is the
// chain of dependent loads (column, then distance) of the longest scan, not
// bytes: on a scale-free graph the hubs are neighbours in vertex order, and
// one wave that scanned the rows of its 64 vertices one after another took
// 1.84 ms (R-MAT, 1,000,003 vertices, 30 M entries, nearly all of it in the
// first few waves).  So rows are split by length.  Up to 64 entries: lane =
// vertex, four entries at a time with the loads issued together.  Longer rows
// go to one list for the whole grid, and a second launch takes them from there,
// so that neighbouring hubs land on different work-groups: a wave per row, 256
// entries per step, and past 2,048 entries the whole work-group, 1,024 entries
// per step.  On the same graph the two launches take 75 + 73 us.
#include <algorithm>

#include "engine.h"

namespace gfr {

struct BfsCloser {
    const int32_t *d;
    __device__ bool reached(int32_t v, int64_t &kv) const
    {
        kv = d[v];
        return kv >= 0;
    }
    __device__ bool closer(int64_t kv, int32_t, int32_t u) const { return (int64_t)d[u] == kv - 1; }
};

struct SsspCloser {
    const uint32_t *d;
    const uint32_t *W;
    __device__ bool reached(int32_t v, int64_t &kv) const
    {
        kv = d[v];
        return d[v] != 0xFFFFFFFFu;
    }
    __device__ bool closer(int64_t kv, int32_t e, int32_t u) const
    {
        const uint32_t du = d[u];
        return (du != 0xFFFFFFFFu) & ((int64_t)du + (int64_t)W[e] == kv);
    }
};

constexpr int32_t PRED_LANE_ROW = 64;     // longest row one lane scans
constexpr int32_t PRED_WAVE_ROW = 2048;   // longest row one wave scans
constexpr int PRED_STAGE = 1024;          // long rows a work-group gathers before it appends them to the list

// Rows of more than PRED_LANE_ROW entries waiting for pred_long: those of up
// to PRED_WAVE_ROW entries from the front of v, the others from its end
// (together at most m / (PRED_LANE_ROW + 1)).
struct PredList {
    int32_t *v;
    uint32_t cap;
    uint32_t *count;   // [0] front, [1] end
};

// Append the staged rows (whole work-group; s_n is 0 afterwards).
__device__ __forceinline__ void pred_flush(const PredList &list, const int32_t *R, const int32_t *s_v, uint32_t *s_n)
{
    __shared__ uint32_t s_big, s_base[2];
    __syncthreads();
    const uint32_t cnt = *s_n;
    if (threadIdx.x == 0) s_big = 0;
    __syncthreads();
    uint32_t slot[PRED_STAGE / GFR_BLOCK];   // place among the big rows, or ~0
#pragma unroll
    for (int k = 0; k < PRED_STAGE / GFR_BLOCK; ++k) {
        const uint32_t i = k * GFR_BLOCK + threadIdx.x;
        slot[k] = ~0u;
        if (i < cnt && R[s_v[i] + 1] - R[s_v[i]] > PRED_WAVE_ROW) slot[k] = atomicAdd(&s_big, 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (cnt > s_big) s_base[0] = atomicAdd(list.count, cnt - s_big);
        if (s_big) s_base[1] = atomicAdd(list.count + 1, s_big);
        *s_n = 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) s_big = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PRED_STAGE / GFR_BLOCK; ++k) {
        const uint32_t i = k * GFR_BLOCK + threadIdx.x;
        if (i >= cnt) continue;
        if (slot[k] == ~0u) list.v[s_base[0] + atomicAdd(&s_big, 1u)] = s_v[i];
        else list.v[list.cap - 1u - (s_base[1] + slot[k])] = s_v[i];
    }
}

template <class T>
__global__ __launch_bounds__(GFR_BLOCK) void pred_kernel(const int32_t *R, const int32_t *C, int32_t n, int32_t src,
                                                         T t, int32_t *pred, PredList list)
{
    __shared__ int32_t s_v[PRED_STAGE];
    __shared__ uint32_t s_n;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    const uint32_t step = gridDim.x * GFR_BLOCK;
    for (uint32_t v0 = blockIdx.x * GFR_BLOCK; v0 < (uint32_t)n; v0 += step) {
        const int32_t v = (int32_t)(v0 + threadIdx.x);
        int32_t p = -1;
        int64_t kv = 0;
        if (v < n && t.reached(v, kv)) {
            if (v == src) {
                p = src;
            } else {
                const uint32_t rb = (uint32_t)R[v], re = (uint32_t)R[v + 1];
                if (re - rb > (uint32_t)PRED_LANE_ROW) {
                    s_v[atomicAdd(&s_n, 1u)] = v;   // at most GFR_BLOCK a turn: room was made below
                } else {
                    for (uint32_t e = rb; e < re; e += 4) {
                        const uint32_t k = min(4u, re - e);
                        int32_t u[4];
#pragma unroll
                        for (uint32_t j = 0; j < 4; ++j) u[j] = C[j < k ? e + j : e];
                        bool hit[4];
#pragma unroll
                        for (uint32_t j = 0; j < 4; ++j)
                            hit[j] = (j < k) & t.closer(kv, (int32_t)(j < k ? e + j : e), u[j]);
                        int32_t f = -1;
#pragma unroll
                        for (int j = 3; j >= 0; --j) f = hit[j] ? u[j] : f;
                        if (f >= 0) {
                            p = f;
                            break;
                        }
                    }
                }
            }
        }
        if (v < n) pred[v] = p;
        if (list.cap) {   // uniform
            __syncthreads();
            if (s_n > (uint32_t)(PRED_STAGE - GFR_BLOCK)) pred_flush(list, R, s_v, &s_n);
            __syncthreads();
        }
    }
    if (list.cap) pred_flush(list, R, s_v, &s_n);
}

// The rows of the list: first the longest, a work-group each, then the rest, a wave each.
template <class T>
__global__ __launch_bounds__(GFR_BLOCK) void pred_long(const int32_t *R, const int32_t *C, T t, int32_t *pred,
                                                       PredList list)
{
    constexpr int EPL = 4;   // entries per lane and step
    __shared__ int32_t s_first;
    const uint32_t nwave = list.count[0], nbig = list.count[1];
    for (uint32_t i = blockIdx.x; i < nbig; i += gridDim.x) {
        const int32_t v = list.v[list.cap - 1u - i];
        int64_t kv;
        t.reached(v, kv);
        const int32_t rb = R[v], re = R[v + 1];
        for (int32_t e0 = rb; e0 < re; e0 += EPL * GFR_BLOCK) {
            if (threadIdx.x == 0) s_first = INT32_MAX;
            __syncthreads();
            int32_t u[EPL];
#pragma unroll
            for (int j = 0; j < EPL; ++j) u[j] = C[min((int64_t)e0 + j * GFR_BLOCK + threadIdx.x, (int64_t)re - 1)];
            int32_t first = INT32_MAX;
#pragma unroll
            for (int j = EPL - 1; j >= 0; --j) {
                const int64_t e = (int64_t)e0 + j * GFR_BLOCK + threadIdx.x;
                if ((e < re) & t.closer(kv, (int32_t)min(e, (int64_t)re - 1), u[j])) first = (int32_t)(e - e0);
            }
            if (first != INT32_MAX) atomicMin(&s_first, first);
            __syncthreads();
            const int32_t f = s_first;
            __syncthreads();
            if (f != INT32_MAX) {
                if (threadIdx.x == 0) pred[v] = C[e0 + f];
                break;
            }
            if (re - e0 <= EPL * GFR_BLOCK) break;   // (e0 stays within 31 bits)
        }
    }
    const int lane = lane_id();
    for (uint32_t i = blockIdx.x * GFR_WAVES + threadIdx.x / 64; i < nwave; i += gridDim.x * GFR_WAVES) {
        const int32_t v = list.v[i];
        int64_t kv;
        t.reached(v, kv);
        const int32_t rb = R[v], re = R[v + 1];
        int32_t found = -1;
        for (int32_t e0 = 0; e0 < re - rb && found < 0; e0 += EPL * 64) {
            int32_t u[EPL];
#pragma unroll
            for (int j = 0; j < EPL; ++j) u[j] = C[rb + min(e0 + j * 64 + lane, re - rb - 1)];
            uint64_t hm[EPL];
#pragma unroll
            for (int j = 0; j < EPL; ++j) {
                const int32_t e = min(e0 + j * 64 + lane, re - rb - 1);
                hm[j] = ballot((e0 + j * 64 + lane < re - rb) & t.closer(kv, rb + e, u[j]));
            }
#pragma unroll
            for (int j = EPL - 1; j >= 0; --j)
                if (hm[j]) found = (int32_t)shfl_u32((uint32_t)u[j], __ffsll((unsigned long long)hm[j]) - 1);
        }
        if (lane == 0) pred[v] = found;
    }
}

size_t pred_scratch_bytes(const Graph &g)
{
    return g.max_deg > PRED_LANE_ROW ? al256(4ull * (size_t)(g.m / (PRED_LANE_ROW + 1) + 1)) + al256(8) : 0;
}

template <class T>
static void run_pred(Ctx &c, Graph &g, int32_t src, T t, int32_t *pred, hipStream_t s)
{
    // the list and its launch only where some row is long (a lattice has none)
    PredList list{nullptr, 0u, nullptr};
    if (g.max_deg > PRED_LANE_ROW) {
        list.cap = (uint32_t)(g.m / (PRED_LANE_ROW + 1) + 1);
        list.v = c.arena.take<int32_t>(list.cap);
        list.count = c.arena.take<uint32_t>(2);
        fill_u32(list.count, 0u, 2, s);
    }
    const int32_t *R = g.R.as<int32_t>(), *C = g.C.as<int32_t>();
    const unsigned need = (unsigned)(((size_t)g.n + GFR_BLOCK - 1) / GFR_BLOCK);
    hipLaunchKernelGGL(pred_kernel<T>, dim3(std::min(need, (unsigned)grid_blocks(c, 8))), dim3(GFR_BLOCK), 0, s, R, C,
                       g.n, src, t, pred, list);
    if (list.cap)
        hipLaunchKernelGGL(pred_long<T>, dim3(grid_blocks(c, 8)), dim3(GFR_BLOCK), 0, s, R, C, t, pred, list);
    GFR_LAUNCH_CHECK();
}

void run_bfs_pred(Ctx &c, Graph &g, int32_t src, const int32_t *depth, int32_t *pred, hipStream_t s)
{
    run_pred(c, g, src, BfsCloser{depth}, pred, s);
}

void run_sssp_pred(Ctx &c, Graph &g, int32_t src, const uint32_t *dist, int32_t *pred, hipStream_t s)
{
    run_pred(c, g, src, SsspCloser{dist, g.W.as<uint32_t>()}, pred, s);
}

}  // namespace gfr
