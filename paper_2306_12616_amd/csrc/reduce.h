// Deterministic wavefront / workgroup reductions (fixed combination order).
#pragma once

#include <hip/hip_runtime.h>

namespace chebdm {

// The butterfly op(v[l], v[l ^ off]) for off = 32, 16, 8, 4, 2, 1, every lane receiving the result, without
// LDS: the first two steps by lane-half and row swaps, then DPP rotations inside the rows of 16
// (after a step the values repeat with period off, so lane l + off / 2 holds what l ^ (off / 2) does).
// Same operations, same bits as with __shfl_xor, at a fraction of the latency.
template <int N>
__device__ __forceinline__ double row_rotate(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x120 + N, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x120 + N, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

template <class Op>
__device__ __forceinline__ double wave_reduce(double v, Op op) {
    {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
        v = op(__builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]),
               __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]));
    }
    {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
        v = op(__builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]),
               __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]));
    }
    v = op(v, row_rotate<8>(v));
    v = op(v, row_rotate<4>(v));
    v = op(v, row_rotate<2>(v));
    return op(v, row_rotate<1>(v));
}

__device__ __forceinline__ double wave_sum(double v) {
    return wave_reduce(v, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ double wave_min(double v) {
    return wave_reduce(v, [](double a, double b) { return fmin(a, b); });
}
__device__ __forceinline__ double wave_max(double v) {
    return wave_reduce(v, [](double a, double b) { return fmax(a, b); });
}

// Sum over a workgroup of NT threads; every thread receives the result.
// smem must hold NT/64 doubles and is reused after a barrier.
template <int NT>
__device__ inline double block_sum(double v, double* smem) {
    static_assert(NT % 64 == 0 && NT <= 1024, "workgroup must be whole wavefronts");
    constexpr int NW = NT / 64;
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) smem[wid] = v;
    __syncthreads();
    double r = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) r += smem[w];
    return r;
}

template <int NT>
__device__ inline double block_min(double v, double* smem) {
    constexpr int NW = NT / 64;
    v = wave_min(v);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) smem[wid] = v;
    __syncthreads();
    double r = smem[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) r = fmin(r, smem[w]);
    return r;
}

template <int NT>
__device__ inline double block_max(double v, double* smem) {
    constexpr int NW = NT / 64;
    v = wave_max(v);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) smem[wid] = v;
    __syncthreads();
    double r = smem[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) r = fmax(r, smem[w]);
    return r;
}

}  // namespace chebdm
