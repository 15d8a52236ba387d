// nearness.h -- how much of a graph's edges stay between neighbouring ids (host
// only, no HIP).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace gfr {

// Share of the entries whose two ends lie in the same aligned run of NEAR_RUN
// ids, from 4,096 entries spread evenly over the columns (1 without entries).
constexpr int32_t NEAR_RUN = 8192;
constexpr double NEAR_SHARE = 0.84;   // from here on a graph counts as numbered along its edges

inline double near_share(int32_t n, int64_t m, const int32_t *R, const int32_t *C)
{
    if (m == 0 || n <= NEAR_RUN) return 1.0;
    const int64_t samples = std::min<int64_t>(m, 4096);
    int64_t near = 0;
    for (int64_t i = 0; i < samples; ++i) {
        const int64_t e = m / samples * i + m % samples * i / samples;
        const int32_t u = (int32_t)(std::upper_bound(R, R + n + 1, (int32_t)e) - R) - 1;   // the row that holds e
        near += u / NEAR_RUN == C[e] / NEAR_RUN;
    }
    return (double)near / (double)samples;
}

}  // namespace gfr
