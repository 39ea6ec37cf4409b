// ff_scan.h — block-wide helpers of the tile sorts shared by the density
// histogram and the tiled particle image.  Each translation unit gets its own
// copy (internal linkage).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace ff {
namespace {

// Exclusive scan over a block of up to 1024 threads (whole wavefronts of 64):
// returns the exclusive prefix of v and writes the block total to *total.
// wsum: 32 words of LDS.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* wsum, uint32_t* total) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, waves = blockDim.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(inc, off, 64);
        if (lane >= off) inc += t;
    }
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    if (wv == 0) {
        uint32_t s = lane < waves ? wsum[lane] : 0u;
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
            const uint32_t t = __shfl_up(s, off, 64);
            if (lane >= off) s += t;
        }
        if (lane < 16) wsum[16 + lane] = s;  // inclusive scan of wave sums
    }
    __syncthreads();
    const uint32_t before = wv ? wsum[16 + wv - 1] : 0u;
    *total = wsum[16 + 15];
    __syncthreads();
    return before + inc - v;
}

// Adds 1 to s[v] for every active lane; returns what the lane's 1 was added
// to.  Lanes that all hit one counter (an ensemble sitting on a fixed point)
// would be served one by one; they add their number once.
__device__ __forceinline__ uint32_t count_one(uint32_t* s, uint32_t v) {
    const uint64_t live = __ballot(1);
    const uint32_t first = __builtin_amdgcn_readfirstlane(v);
    if (__ballot(v != first) != 0) return atomicAdd(&s[v], 1u);
    const uint32_t below =
        __builtin_amdgcn_mbcnt_hi((uint32_t)(live >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)live, 0u));
    uint32_t base = 0;
    if (below == 0) base = atomicAdd(&s[first], (uint32_t)__popcll(live));
    return (uint32_t)__builtin_amdgcn_readfirstlane(base) + below;
}

}  // namespace
}  // namespace ff
