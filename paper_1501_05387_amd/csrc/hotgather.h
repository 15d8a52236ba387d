// hotgather.h -- segmented gather-reduce over the whole graph for rankings that
// iterate to convergence on scale-free graphs:
//     S(i) = sum over the neighbours u of entry i's vertex of x(u),
// FP64 sums of a table x of T, per entry of the whole-graph queue.
//
// A sweep over the CSR is bound by its random reads of x (gather.h): R-MAT s22
// reads 128 M entries of a 16.8 MB table at 160 G/s, because a line of the
// table holds 32 vertices of very different degree, so that L2 (4 MB per XCD)
// is full of values that are hardly read.  Here the table is kept in order of
// degree, and the columns of the graph are renumbered to match (RankedCols,
// made once per graph).  The first H values, which most edges name, are copied
// to LDS by every work-group; the next ones share their lines with others as
// hot as they are.
//
// One wave takes 256 consecutive edges at a time, four per lane, and needs no
// other wave: the list starts are a bitmap over the edges and the entry that
// holds a chunk's first edge is stored, so all of a chunk's reads but the
// gathers themselves are independent and are issued one chunk ahead.  Sums are
// formed by a segmented scan in registers in a fixed order, as in gather.h.
//
// A sweep of R-MAT s22 takes 0.41 ms (0.80 over the CSR): 61 M L2 requests, of
// which 11 M miss; half the waves per CU take as long, so their rate, not
// latency, is what is left.  Tables of 32, 72, 128 and 152 KB in LDS (the first
// two with two work-groups per CU): 0.55, 0.51, 0.47 and 0.45 ms before the
// columns were read ahead.
#pragma once

#include "device.h"
#include "engine.h"
#include "gather.h"

namespace gfr {

constexpr int HG_BLOCK = 1024;      // one work-group per CU: LDS is the table's
constexpr uint32_t HG_CH = 256;     // edges a wave takes at a time
constexpr int HG_HOT_BYTES = 152 * 1024;

// What the kernels read of a graph with ranked columns.
struct HotGraph {
    const int32_t *C;          // position in the table (nf + 1 values) of each edge's target, padded to whole chunks
    const uint32_t *starts;    // bit e: a list starts at edge e (one chunk of padding)
    const int32_t *entry;      // [nch + 1] entry of the whole-graph queue that holds edge c * HG_CH
    const uint32_t *off;       // first edge of each entry
    uint32_t nf, mf, nch;
};

template <class T>
__global__ __launch_bounds__(HG_BLOCK) void gather_hot(HotGraph g, const T *table, double *sum, GatherScratch gs,
                                                       const uint32_t *stop)
{
    constexpr uint32_t H = HG_HOT_BYTES / sizeof(T);
    __shared__ T s_hot[H];
    if (*stop) return;
    for (uint32_t i = threadIdx.x; i < min(H, g.nf + 1u); i += HG_BLOCK) s_hot[i] = table[i];
    __syncthreads();
    typedef int vec4 __attribute__((ext_vector_type(4)));
    struct Chunk {
        vec4 col;
        T far[4];
        uint32_t word;
        int32_t base;
    };
    const uint32_t cold = min(H, g.nf - 1u);   // read by lanes that have no use for it: one address
    const int lane = lane_id();
    const uint32_t k = lane * 4u;
    const uint32_t nwaves = gridDim.x * (HG_BLOCK / 64);
    uint32_t c = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * (HG_BLOCK / 64) + threadIdx.x / 64));
    if (c >= g.nch) return;
    // (past the last chunk: the last one again, not summed; a branch around
    // the loads would have to wait for them where it joins)
    auto columns = [&](Chunk &x, uint32_t at) __attribute__((always_inline)) {
        at = min(at, g.nch - 1u);
        // read once, so not kept in L2 (without the hint 322 us against 314, averaged over all launches of a call,
        // those after its end among them)
        x.col = __builtin_nontemporal_load((const vec4 *)(g.C + (size_t)at * HG_CH + k));
        x.word = g.starts[at * (HG_CH / 32) + k / 32];
        x.base = g.entry[at];
        asm volatile("" ::: "memory");   // issued here, not where it is first used
    };
    auto gathers = [&](Chunk &x) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) x.far[j] = table[(uint32_t)x.col[j] >= H ? (uint32_t)x.col[j] : cold];
        asm volatile("" ::: "memory");
    };
    auto sums = [&](const Chunk &x, uint32_t at) __attribute__((always_inline)) {
        const uint32_t e0 = at * HG_CH;
        double val[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t u = (uint32_t)x.col[j];
            const T near = s_hot[u < H ? u : 0u];
            const double v = (double)(u < H ? near : x.far[j]);
            val[j] = e0 + k + j < g.mf ? v : 0.0;
        }
        const uint32_t starts = x.word >> (k & 31u) & 15u;
        // entry of the edge before this lane's first one
        uint32_t before = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) before += lanes_below(ballot(starts >> j & 1u));
        int ent = x.base + (int)before - (int)(__builtin_amdgcn_readfirstlane((int)starts) & 1);
        double head = 0.0, acc = 0.0;
        bool has = false;
        int ended = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (starts >> j & 1u) {
                if (!has) {
                    head = acc;
                    ended = ent;
                    has = true;
                } else {
                    sum[ent] = acc;
                }
                ++ent;
                acc = 0.0;
            }
            acc += val[j];
        }
        double open = acc;
        uint32_t any = has;
        seg_scan(open, any);
        const double in = dpp_f64<0x138, 0xF>(open);   // wave_shr:1
        const uint32_t in_any = dpp_u32<0x138, 0xF>(any);
        if (has && ended >= x.base) {   // (nothing ends at a start on the chunk's first edge)
            if (in_any) sum[ended] = in + head;
            else gs.pfirst[at] = in + head;
        }
        if (lane == 63) {   // the list open at the chunk's end
            if (any) {      // complete, unless the fix-up finds that it goes on
                sum[ent] = open;
                gs.plast[at] = open;
            } else {
                gs.pfirst[at] = open;
            }
        }
    };
    // One chunk is summed while the gathers of the next and the columns of the
    // one after are under way.  Nothing in the loop may wait for a younger load:
    // loads return in order, so that would be a wait for the gathers too.
    Chunk a, b;
    columns(a, c);
    columns(b, c + nwaves);
    gathers(a);
    for (;;) {
        gathers(b);
        sums(a, c);
        columns(a, c + 2 * nwaves);
        c += nwaves;
        if (c >= g.nch) break;
        gathers(a);
        sums(b, c);
        columns(b, c + 2 * nwaves);
        c += nwaves;
        if (c >= g.nch) break;
    }
}

// The lists that cross chunks: one lane per chunk in which such a list starts;
// lists of many chunks are summed by the whole wave.
static __global__ __launch_bounds__(GFR_BLOCK) void gather_hot_fixup(HotGraph g, double *sum, GatherScratch gs,
                                                                     const uint32_t *stop)
{
    constexpr uint32_t LANE_CHUNKS = 16;
    if (*stop) return;
    const int lane = lane_id();
    for (uint32_t c0 = (blockIdx.x * GFR_WAVES + threadIdx.x / 64) * 64u; c0 < g.nch; c0 += gridDim.x * GFR_BLOCK) {
        const uint32_t c = c0 + lane;
        uint32_t more = 0;   // chunks after c
        int32_t i = 0;
        if (c + 1 < g.nch && !(g.starts[(c + 1) * (HG_CH / 32)] & 1u)) {
            const uint4 *w = (const uint4 *)(g.starts + c * (HG_CH / 32));
            const uint4 a = w[0], b = w[1];
            if (a.x | a.y | a.z | a.w | b.x | b.y | b.z | b.w) {
                i = g.entry[c + 1];
                const uint32_t end = (uint32_t)i + 1u < g.nf ? g.off[i + 1] : g.mf;
                more = (end - 1u) / HG_CH - c;
            }
        }
        if (more && more <= LANE_CHUNKS) {
            double acc = gs.plast[c];
            for (uint32_t j = 1; j <= more; ++j) acc += gs.pfirst[c + j];
            sum[i] = acc;
        }
        uint64_t big = ballot(more > LANE_CHUNKS);
        while (big) {
            const int src = __ffsll((unsigned long long)big) - 1;
            big &= big - 1;
            const uint32_t cs = c0 + src, ms = shfl_u32(more, src);
            double acc = lane == 0 ? gs.plast[cs] : 0.0;
            for (uint32_t j = 1 + lane; j <= ms; j += 64) acc += gs.pfirst[cs + j];
            acc = wave_sum_f64(acc);
            if (lane == src) sum[i] = acc;
        }
    }
}

// The graph's ranked columns, made on first use (queued on s and waited for);
// null where they do not pay or do not fit device memory: the caller sweeps
// the CSR then.
const RankedCols *ranked_cols(Ctx &c, Graph &g, hipStream_t s);
HotGraph hot_graph(const Graph &g, const RankedCols &r);

}  // namespace gfr
