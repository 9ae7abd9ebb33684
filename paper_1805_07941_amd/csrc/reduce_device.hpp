// The ends of the max |.| reductions: what a workgroup does with its maximum.
#pragma once
#include "dfq_device.hpp"

namespace dfq {

constexpr int kBlock = 256;

// The result of one of `sharers` workgroups that raise the same word.  A single one stores it, and nobody clears the word first;
// up to one per compute unit send their atomics straight away (100000 values, 98 workgroups: 5.1 us, with a read before 5.6); of many, most see by a
// read that theirs is no news - the maximum only grows - and spare the word the atomic.
__device__ __forceinline__ void raise_to(uint32_t *out, uint32_t m, unsigned sharers)
{
    if (sharers == 1) *out = m;
    else if (sharers <= 256 || m > __hip_atomic_load(out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(out, m);
}

__device__ __forceinline__ void block_max_to(uint32_t v, uint32_t *out)
{
    __shared__ uint32_t part[kBlock / kWave];
    v = wave_max_u32(v);
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t m = part[0];
#pragma unroll
        for (int i = 1; i < kBlock / kWave; i++) m = max(m, part[i]);
        raise_to(out, m, gridDim.x);
    }
}

__device__ __forceinline__ uint32_t float_magnitude(float v)
{
    const float a = fabsf(v);
    return a == a ? __float_as_uint(a) : 0u;          // NaN elements are skipped
}

__device__ __forceinline__ uint32_t magnitude(int v, int relu)
{
    return v >= 0 ? (uint32_t)v : (relu ? 0u : (uint32_t)0 - (uint32_t)v);
}

}  // namespace dfq
