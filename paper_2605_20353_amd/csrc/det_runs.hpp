// Positions in the sorted (row, sample) pairs of the bit-reproducible form.  A
// call may have up to 2^32 - 1 pairs, so that a position fits 32 bits but a
// position plus a batch need not.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gcp {

// Slice `i` of `slices` (4 or more) of the run [b, e), e > b: equal numbers of
// whole batches (`batch` a power of two up to 64; the last slices may be short
// or empty), fixed by the run's length alone.
__host__ __device__ inline void det_slice(uint32_t b, uint32_t e, uint32_t slices, uint32_t i, uint32_t batch,
                                          uint32_t& lo, uint32_t& hi)
{
    const uint32_t len = e - b;
    const uint32_t per = ((len - 1) / slices + batch) & ~(batch - 1);
    const uint64_t at = (uint64_t)per * i;
    lo = at < len ? b + (uint32_t)at : e;
    hi = e - lo > per ? lo + per : e;
}

// Pairs of the batch at `at`.  A walk that goes on by this number ends at e,
// where one that goes on by whole batches may pass 2^32 and never end.
__host__ __device__ inline uint32_t det_batch(uint32_t at, uint32_t e, uint32_t batch)
{
    return e - at < batch ? e - at : batch;
}

// The position that lane `lane` of the batch at `at` reads: its pair, or past
// the run's end the run's last one (or, where at + lane passes 2^32, an earlier
// one: read ahead, never used).
__host__ __device__ inline uint32_t det_lane(uint32_t at, uint32_t e, uint32_t lane)
{
    return at + lane < e - 1 ? at + lane : e - 1;
}

}  // namespace gcp
