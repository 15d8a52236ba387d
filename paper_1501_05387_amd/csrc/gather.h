// gather.h -- load-balanced segmented gather-reduce over a frontier queue.
//
// For every entry i of a FrontierQ (vertex v_i, neighbour list starting at
// row_i, edge offset off_i in the concatenated lists) compute
//     S_i = sum over the neighbours u of v_i, in CSR order, of op(u)
// in FP64, then call fin(v_i, S_i) exactly once.  This is the advance step of
// Sec. 4.1 with a fused "compute" (Sec. 4.3), in the load-balanced
// partitioning form of Sec. 4.4: each work-group takes an equal slice of
// edges, so one hub's list is spread over many work-groups while short lists
// are packed together.
//
// What bounds a sweep of the whole graph is the rate of its random gathers
// (L2 and MALL requests), so everything around them is kept short and in
// registers: one lane takes four consecutive edges, list starts are bits in
// LDS (a lane finds its entry by a population count, not by a search), and the
// sums are formed by a segmented scan over the wave.  Values staged in LDS,
// searched for per edge and summed one short list per lane took 0.88 + 0.03 ms
// (sweep and fix-up) per PageRank iteration on R-MAT s22 (128 M edges); this form
// takes 0.80 + 0.01.
// Lists that cross chunk boundaries leave partial sums that a second, tiny
// kernel combines in chunk order.  For a fixed queue layout every sum is formed
// in a fixed order, so results are reproducible run to run.
#pragma once

#include "device.h"

namespace gfr {

struct GatherScratch {
    double *pfirst;   // per chunk: partial of the entry continuing into it
    double *plast;    // per chunk: partial of the entry starting in it and continuing out
};

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double x)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint64_t lo = dpp_u32<CTRL, ROWS>((uint32_t)b), hi = dpp_u32<CTRL, ROWS>((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(hi << 32 | lo));
}

template <int CTRL, int ROWS>
__device__ __forceinline__ void seg_scan_step(double &open, uint32_t &any)
{
    const double o = dpp_f64<CTRL, ROWS>(open);
    const uint32_t oa = dpp_u32<CTRL, ROWS>(any);
    open = any ? open : o + open;
    any |= oa;
}

// open: sum of what each lane holds of the list open at its end; any: a list
// starts in the lane.  Afterwards open reaches back to the list's start or the
// wave's, and any says which.
__device__ __forceinline__ void seg_scan(double &open, uint32_t &any)
{
    seg_scan_step<0x111, 0xF>(open, any);   // row_shr:1, :2, :4, :8
    seg_scan_step<0x112, 0xF>(open, any);
    seg_scan_step<0x114, 0xF>(open, any);
    seg_scan_step<0x118, 0xF>(open, any);
    seg_scan_step<0x142, 0xA>(open, any);   // row_bcast:15 into rows 1 and 3
    seg_scan_step<0x143, 0xC>(open, any);   // row_bcast:31 into rows 2 and 3
}

template <int CH, class Op, class Fin>
__global__ __launch_bounds__(GFR_BLOCK) void gather_chunks(FrontierQ q, const uint32_t *nf_p,
                                                           const uint32_t *mf_p, const int32_t *C,
                                                           Op op, Fin fin, GatherScratch gs,
                                                           const uint32_t *stop, QueueAt at = QueueAt{nullptr})
{
    constexpr int EPL = 4;   // consecutive edges per lane
    static_assert(CH == GFR_BLOCK * EPL && CH / 32 <= 64, "a chunk is four edges per thread");
    if (*stop) return;
    const uint32_t nf = *nf_p, mf = *mf_p;
    const uint32_t nchunks = (mf + CH - 1) / CH;
    if (blockIdx.x >= nchunks) return;
    q = at(q);
    __shared__ uint32_t s_flag[CH / 32];    // bit k: a list starts at edge k of the chunk
    __shared__ int32_t s_delta[CH + 1];     // per entry: its place in C less its edge offset
    __shared__ int32_t s_v[CH + 1];
    __shared__ double s_carry[GFR_WAVES];   // per wave: sum of the list open at its end
    __shared__ uint32_t s_has[GFR_WAVES];   // per wave: a list starts in it
    const int wave = threadIdx.x / 64, lane = lane_id();
    for (uint32_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const uint32_t e0 = c * CH;
        const uint32_t e1 = min(e0 + (uint32_t)CH, mf);
        const int s = q.part[c];
        const int t = (c + 1 < nchunks) ? q.part[c + 1] : (int)nf - 1;
        const int cnt = t - s + 1;
        __syncthreads();
        if (threadIdx.x < CH / 32) s_flag[threadIdx.x] = 0;
        __syncthreads();
        for (int i = threadIdx.x; i < cnt; i += GFR_BLOCK) {
            const uint32_t off = q.off[s + i];
            s_delta[i] = q.row[s + i] - (int32_t)off;
            s_v[i] = q.v[s + i];
            // (the first list may start before the chunk, the last one at its end)
            if (off >= e0 && off < e1) atomicOr(&s_flag[(off - e0) >> 5], 1u << ((off - e0) & 31));
        }
        __syncthreads();
        // starts before this lane's edges
        const uint32_t k = threadIdx.x * EPL;
        const uint32_t word = s_flag[lane & (CH / 32 - 1)];
        const uint32_t incl = wave_incl_scan(lane < CH / 32 ? __popc(word) : 0u);
        const uint32_t mine = shfl_u32(word, k >> 5);
        uint32_t before = shfl_u32(incl, k >> 5) - __popc(mine) + __popc(mine & ((1u << (k & 31)) - 1u));
        before -= s_flag[0] & 1u;   // entry 0 counts as started
        const uint32_t starts = mine >> (k & 31) & ((1u << EPL) - 1u);
        int ent[EPL];
        int32_t u[EPL];
#pragma unroll
        for (int j = 0; j < EPL; ++j) {
            ent[j] = (int)(before + __popc(starts & ((2u << j) - 1u)));
            const uint32_t e = min(e0 + k + j, e1 - 1u);   // past the end: the last edge again (and its entry), not added
            u[j] = C[(int32_t)e + s_delta[ent[j]]];
        }
        double val[EPL];
#pragma unroll
        for (int j = 0; j < EPL; ++j) val[j] = op(u[j]);
        // the lane's own lists: head = what belongs to the list open before it
        double head = 0.0, acc = 0.0;
        bool has = false;
        int ended = 0;   // the entry that ends at the lane's first start
#pragma unroll
        for (int j = 0; j < EPL; ++j) {
            if (starts >> j & 1u) {
                if (!has) {
                    head = acc;
                    ended = ent[j] - 1;
                    has = true;
                } else {
                    fin(s_v[ent[j] - 1], acc);
                }
                acc = 0.0;
            }
            if (e0 + k + j < e1) acc += val[j];
        }
        // sum of the list open at each lane's end, back to its start or the wave's
        double open = acc;
        uint32_t any = has;
        seg_scan(open, any);
        const double in = dpp_f64<0x138, 0xF>(open);   // wave_shr:1
        const uint32_t in_any = dpp_u32<0x138, 0xF>(any);
        if (lane == 63) {
            s_carry[wave] = open;
            s_has[wave] = any;
        }
        __syncthreads();
        // of the waves before
        double wsum = 0.0;
        uint32_t wany = 0;
        for (int w = 0; w < wave; ++w) {
            wsum = s_has[w] ? s_carry[w] : wsum + s_carry[w];
            wany |= s_has[w];
        }
        if (has && ended >= 0) {   // (nothing ends at a start on the chunk's first edge)
            const double sum = (in_any ? in : wsum + in) + head;
            if (in_any | wany) fin(s_v[ended], sum);
            else gs.pfirst[c] = sum;
        }
        if (threadIdx.x == GFR_BLOCK - 1) {   // the list open at the chunk's end
            const double sum = any ? open : wsum + open;
            const int i = (int)before + __popc(starts);
            const uint32_t end = s + i + 1 < (int)nf ? q.off[s + i + 1] : mf;
            if (!(any | wany)) gs.pfirst[c] = sum;
            else if (end <= e1) fin(s_v[i], sum);
            else gs.plast[c] = sum;
        }
    }
}

// One lane per chunk: if the chunk's last entry starts in it and continues
// past its end, add the partials of the following chunks in order.
template <int CH, class Fin>
__global__ __launch_bounds__(GFR_BLOCK) void gather_fixup(FrontierQ q, const uint32_t *nf_p,
                                                          const uint32_t *mf_p, Fin fin,
                                                          GatherScratch gs, const uint32_t *stop,
                                                          QueueAt at = QueueAt{nullptr})
{
    if (*stop) return;
    const uint32_t nf = *nf_p, mf = *mf_p;
    const uint32_t nchunks = (mf + CH - 1) / CH;
    if (blockIdx.x * GFR_BLOCK >= nchunks) return;
    q = at(q);
    for (uint32_t c = blockIdx.x * GFR_BLOCK + threadIdx.x; c < nchunks; c += gridDim.x * GFR_BLOCK) {
        const uint32_t e0 = c * CH, e1 = min(e0 + (uint32_t)CH, mf);
        const int t = (c + 1 < nchunks) ? q.part[c + 1] : (int)nf - 1;
        const uint32_t ot = q.off[t];
        const uint32_t endt = (t + 1 < (int)nf) ? q.off[t + 1] : mf;
        if (ot < e0 || ot >= e1 || endt <= e1) continue;  // not the head of a split list
        double acc = gs.plast[c];
        const uint32_t last = (endt - 1u) / CH;   // the chunk it ends in
        uint32_t c2 = c + 1;
        for (; c2 + 8 <= last + 1; c2 += 8) {   // a hub's list spans hundreds: eight loads together
            double p[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) p[j] = gs.pfirst[c2 + j];
#pragma unroll
            for (int j = 0; j < 8; ++j) acc += p[j];
        }
        for (; c2 <= last; ++c2) acc += gs.pfirst[c2];
        fin(q.v[t], acc);
    }
}

// Visit every edge (v_i -> u) of the queue once, load-balanced over edges:
// op(u, v_i) runs on one lane per edge.  Used where the per-edge work has no
// reduction (the 2-hop pushes).
template <int CH, class Op>
__global__ __launch_bounds__(GFR_BLOCK) void for_each_edge(FrontierQ q, const uint32_t *nf_p,
                                                           const uint32_t *mf_p, const int32_t *C,
                                                           Op op)
{
    const uint32_t nf = *nf_p, mf = *mf_p;
    const uint32_t nchunks = (mf + CH - 1) / CH;
    __shared__ uint32_t s_off[CH + 1];
    __shared__ int32_t s_row[CH + 1];
    __shared__ int32_t s_v[CH + 1];
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
            s_v[i] = q.v[s + i];
        }
        __syncthreads();
        for (uint32_t k = 0; k < (uint32_t)CH; k += GFR_BLOCK) {
            const uint32_t e = e0 + k + threadIdx.x;
            const bool valid = e < e1;
            int32_t u = 0, v = 0;
            if (valid) {
                const int i = upper_index(s_off, 0, cnt - 1, e);
                u = C[s_row[i] + (int32_t)(e - s_off[i])];
                v = s_v[i];
            }
            op(valid, u, v);   // called by every lane (converged), valid marks real edges
        }
    }
}

}  // namespace gfr
