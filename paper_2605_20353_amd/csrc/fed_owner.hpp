// Threads of a row-block owner workgroup in the batched federated round.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace gcp {

// `blocks` workgroups, one per row block, expect `total` entries together and
// `largest` in the fullest block; places[i] of them run at once with 1024 >> i
// threads.  A workgroup's wavefronts share its entries, so that it ends after
// entries / wavefronts steps, and workgroups that find no place start after
// others: 1024 threads, or fewer where all workgroups then start at once and
// the fullest block does not hold the launch up by more than a quarter.  (16
// clients of 5000 x 5000 x 500 blocks at rank 32: 640 equal row blocks, 512
// places with 1024 threads, 925 us a round with 512 threads and 949 with 1024.
// 8 clients of 4500 x 200 x 350 in double at rank 24: 39 row blocks a client, 10000
// entries in three of them, 830 in the others, 256 places: 1040 us a round with
// 512 threads, 768 with 1024.)
inline int fed_owner_threads(int64_t blocks, double total, double largest, const int64_t (&places)[3])
{
    auto steps = [&](int i) {
        const double rounds = (double)((blocks + std::max<int64_t>(1, places[i]) - 1) / std::max<int64_t>(1, places[i]));
        return std::max(largest, rounds * total / (double)std::max<int64_t>(1, blocks)) / (double)(16 >> i);
    };
    for (int i = 0; i < 3; ++i)
        if (blocks <= places[i]) return steps(i) <= 1.25 * steps(0) ? 1024 >> i : 1024;
    return 1024;
}

}  // namespace gcp
