// Device code shared by the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "grim_internal.h"

namespace grim {

// x of lane ^ 16 and of lane ^ 32: the swaps leave both rows (halves) of each pair
// in every lane of the pair.
__device__ __forceinline__ uint32_t lane_xor16(uint32_t x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return (threadIdx.x & 16) ? r[0] : r[1];
}

__device__ __forceinline__ uint32_t lane_xor32(uint32_t x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return (threadIdx.x & 32) ? r[0] : r[1];
}

template <int CTRL>
__device__ __forceinline__ uint32_t lane_dpp(uint32_t x)
{
    return __builtin_amdgcn_mov_dpp(x, CTRL, 0xF, 0xF, true);
}

// x of lane ^ m, for m a power of two or one less than one (known at compile time
// after unrolling), with every lane active: DPP moves within rows of 16 lanes,
// gfx950's row and half-wavefront swaps across them.  No LDS crossbar, whose
// round trip (and, in the sorts, whose rate) these chains of exchanges waited on.
__device__ __forceinline__ uint32_t lane_xor(uint32_t x, int m)
{
    constexpr int kHalfMirror = 0x141, kMirror = 0x140, kReverse4 = 0x1B;   // ^ 7, ^ 15, ^ 3
    switch (m) {
    case 1: return lane_dpp<0xB1>(x);                 // quad_perm 1,0,3,2
    case 2: return lane_dpp<0x4E>(x);                 // quad_perm 2,3,0,1
    case 3: return lane_dpp<kReverse4>(x);
    case 4: return lane_dpp<kReverse4>(lane_dpp<kHalfMirror>(x));
    case 7: return lane_dpp<kHalfMirror>(x);
    case 8: return lane_dpp<0x128>(x);                // row_ror 8
    case 15: return lane_dpp<kMirror>(x);
    case 16: return lane_xor16(x);
    case 31: return lane_xor16(lane_dpp<kMirror>(x));
    case 32: return lane_xor32(x);
    case 63: return lane_xor32(lane_xor16(lane_dpp<kMirror>(x)));
    default: return __shfl_xor(x, m);
    }
}

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
