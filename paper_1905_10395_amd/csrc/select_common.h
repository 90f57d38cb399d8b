// Keys and wavefront reductions of the leader selection.
//
// A loss and its worker index are packed into one 64-bit key whose unsigned
// order is (loss ascending, index ascending), so a plain integer minimum is
// the argmin with the required tie-break (lowest index; NaN counts as +infinity).
#pragma once

#include "common.h"

namespace lsgd {

__device__ __forceinline__ uint64_t loss_key(float v, int idx)
{
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) u = 0x7F800000u; // NaN -> +inf
    if (u == 0x80000000u) u = 0u;                         // -0 ties with +0
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);       // monotone map to unsigned
    return ((uint64_t)u << 32) | (uint32_t)idx;
}

__device__ __forceinline__ uint64_t shfl_up_u64(uint64_t v, int d)
{
    uint32_t lo = __shfl_up((uint32_t)v, d, kWave);
    uint32_t hi = __shfl_up((uint32_t)(v >> 32), d, kWave);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int d)
{
    uint32_t lo = __shfl_xor((uint32_t)v, d, kWave);
    uint32_t hi = __shfl_xor((uint32_t)(v >> 32), d, kWave);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t wave_min_u64(uint64_t k)
{
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        uint64_t o = shfl_xor_u64(k, d);
        k = o < k ? o : k;
    }
    return k;
}

__device__ __forceinline__ void write_plan_rows(int tid, int nthreads, int W, int G, const int32_t* group_of, const int32_t* lead,
                                                const int32_t* glead, const int32_t* refreshed, RowPlan* plan)
{
    for (int i = tid; i < W; i += nthreads) {
        const int j = group_of[i];
        RowPlan r;
        r.ll = lead[j]; r.gl = glead[0]; r.freshL = refreshed[j]; r.freshG = refreshed[G]; r.j = j;
        r.pad[0] = r.pad[1] = r.pad[2] = 0;
        plan[i] = r;
    }
}

} // namespace lsgd
