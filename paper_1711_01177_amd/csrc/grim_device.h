// Device code shared by the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "grim_internal.h"

namespace grim {

// Read that owns pair p: the last r with cand_off[r] <= p, found by the whole
// wave 64 ways at a time (one memory round trip per factor of 64 reads).
__device__ __forceinline__ uint64_t wave_read_of(const uint64_t *__restrict__ cand_off,
                                                 uint64_t n_reads, uint64_t p, int lane)
{
    uint64_t lo = 0, n = n_reads;   // the answer is in [lo, lo + n)
    while (n > 1) {
        const uint64_t step = (n + kWave - 1) / kWave;
        const uint64_t i = lo + (uint64_t)lane * step;
        const bool le = (uint64_t)lane * step < n && cand_off[i] <= p;
        const uint64_t m = __ballot(le);
        // highest lane at or below p (lane 0's read when none is)
        const int h = m ? 63 - __builtin_clzll(m) : 0;
        const uint64_t left = n - (uint64_t)h * step;
        lo += (uint64_t)h * step;
        n = left < step ? left : step;
    }
    return lo;
}

}  // namespace grim
