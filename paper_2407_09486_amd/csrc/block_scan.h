// Device pieces shared by the kernels that walk the streams' offsets.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace enova {

namespace {

// Steps of the reference prefix of a stream of T steps.
__device__ __forceinline__ int64_t ref_len_dev(float ref_frac, int64_t T)
{
    return static_cast<int64_t>(floor(static_cast<double>(ref_frac) * static_cast<double>(T)));
}

// Exclusive prefix of each thread's value over the block's NT threads, and the block's total: a
// shuffle scan in each wave, then the wave totals in wave order (integer sums: any order gives
// the same). Two barriers; one thread walking the 1024 sums in LDS took 10 of the kernel's 13 us.
template <int NT>
__device__ __forceinline__ int64_t block_scan_excl(int64_t v, int64_t *wsum, int64_t &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int64_t o = __shfl_up(inc, off);
        if (lane >= off)
            inc += o;
    }
    if (lane == 63)
        wsum[wave] = inc;
    __syncthreads();
    int64_t base = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        const int64_t t = wsum[w];
        base += w < wave ? t : 0;
        sum += t;
    }
    total = sum;
    return base + inc - v;
}

}  // namespace

}  // namespace enova
