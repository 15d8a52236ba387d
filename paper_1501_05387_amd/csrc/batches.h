// batches.h -- how many launches a level loop queues before the host looks at
// the control block again (host only, no HIP).
//
// A launch that finds the solve ended costs 3.5 to 5 us (a PageRank iteration is
// four of them), a look about 30 us: 10 to 15 of waiting, and the queue runs dry
// meanwhile.
#pragma once

#include <stdint.h>

namespace gfr {

// The next batch after `launched` launches that were not enough, where an
// earlier solve gave the size of the first batch: a quarter of them, at least
// eight and at most 256 (as many again while there are fewer than eight).  A
// traversal a few levels longer than the last one would otherwise queue its
// whole length again.
constexpr int32_t next_batch(int64_t launched)
{
    if (launched < 8) return (int32_t)launched;
    const int64_t quarter = launched / 4;
    return (int32_t)(quarter < 8 ? 8 : quarter > 256 ? 256 : quarter);
}

// The same where nothing is known beforehand (PageRank and its kin, from eight
// on): doubling in two halves, 8, 8, 8, 16, 16, 32, 32, ...  Doubling at once
// queues up to as many iterations in vain as were needed, quarters look too often.
// PageRank on a path of 20,000 vertices, 9, 24, 25, 56 and 57 iterations: 308,
// 476, 594, 1,085 and 1,114 us in quarters; 376, 442, 792, 948 and 1,628 in
// batches of 8, 16, 32, 64.
constexpr int32_t next_batch_unknown(int64_t launched)
{
    if (launched < 8) return (int32_t)launched;
    int64_t power = 16;
    while (2 * power <= launched + 8) power *= 2;
    return (int32_t)(power / 2 > 256 ? 256 : power / 2);
}

}  // namespace gfr
