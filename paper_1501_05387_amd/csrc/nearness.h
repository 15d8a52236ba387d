// nearness.h -- how much of a graph's edges stay between neighbouring ids (host
// only, no HIP).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace gfr {

// Share of the entries whose two ends lie in the same aligned run of NEAR_RUN
// ids, from 256 to 1,024 entries spread over the columns (1 without entries), one
// anywhere in each of as many pieces: even rows repeat every few entries.
// The row of an entry is searched for around where it would be with even rows:
// the load of a graph of 39,000 vertices takes 270 us, and 4,096 searches of the
// whole array took 100.
constexpr int32_t NEAR_RUN = 8192;
constexpr double NEAR_SHARE = 0.84;   // from here on a graph counts as numbered along its edges

inline double near_share(int32_t n, int64_t m, const int32_t *R, const int32_t *C)
{
    if (m == 0 || n <= NEAR_RUN) return 1.0;
    const int64_t samples = std::min<int64_t>(m, std::max(256, std::min(1024, n / 128)));
    int64_t near = 0;
    for (int64_t i = 0; i < samples; ++i) {
        const int64_t e0 = i * m / samples, e1 = (i + 1) * m / samples;
        const int64_t e = e0 + (int64_t)((uint32_t)i * 2654435769u) % (e1 - e0);
        int64_t lo = std::min<int64_t>(n - 1, (int64_t)((double)e / (double)m * n)), hi = lo + 1;
        for (int64_t step = 16; R[lo] > e; step *= 4) lo = std::max<int64_t>(0, lo - step);    // (R[0] is 0)
        for (int64_t step = 16; R[hi] <= e; step *= 4) hi = std::min<int64_t>(n, hi + step);   // (R[n] is m)
        const int32_t u = (int32_t)(std::upper_bound(R + lo, R + hi + 1, (int32_t)e) - R) - 1;   // the row that holds e
        near += u / NEAR_RUN == C[e] / NEAR_RUN;
    }
    return (double)near / (double)samples;
}

}  // namespace gfr
