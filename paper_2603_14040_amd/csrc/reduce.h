// Deterministic block reductions with wave64 shuffles (CDNA wavefront = 64 lanes).
#pragma once
#include <hip/hip_runtime.h>

namespace tph {

// v of lane l + 32, + 16 (in the lower half, the even rows) by lane swaps, and
// of lane l +- CTRL's rotation within its row of 16: register moves, no LDS.
__device__ __forceinline__ double wave_add_halves(double v) {
    const long long b = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) + __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double wave_add_rows(double v) {
    const long long b = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) + __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}
template <int CTRL>
__device__ __forceinline__ double row16_rotate(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Sum over the 16 lanes of a DPP row: lane 0 of the row holds
// ((v0 + v8) + (v4 + v12)) + ..., the tree of halving distances.
__device__ __forceinline__ double row16_sum(double v) {
    v += row16_rotate<0x128>(v);          // row_ror:8, 4, 2, 1
    v += row16_rotate<0x124>(v);
    v += row16_rotate<0x122>(v);
    v += row16_rotate<0x121>(v);
    return v;
}

// Sum over a wave in the tree of halving distances 32, 16, .. 1 (as a chain of
// __shfl_down gives lane 0, whose 12 LDS permutes it replaces): valid in lane 0.
__device__ __forceinline__ double wave_sum(double v) { return row16_sum(wave_add_rows(wave_add_halves(v))); }

// Sums over a block of up to 1024 threads of N values each, value v valid in
// thread v: one barrier whatever N.  All threads must call it; part holds 16 N
// doubles.
template <int N>
__device__ __forceinline__ double block_sums(const double (&a)[N], double* part) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int v = 0; v < N; ++v) {
        const double s = wave_sum(a[v]);
        if ((tid & 63) == 0) part[(tid >> 6) * N + v] = s;
    }
    __syncthreads();
    double t = 0.0;
    if (tid < N) {
        const int nw = (blockDim.x + 63) >> 6;
        for (int w = 0; w < nw; ++w) t += part[w * N + tid];
    }
    return t;
}

// Sum over a block of up to 1024 threads; the result is valid in thread 0.
// All threads of the block must call it (it synchronises twice).
__device__ __forceinline__ double block_sum(double v) {
    __shared__ double part[16];
    const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
    const int nthr = blockDim.x * blockDim.y * blockDim.z;
    v = wave_sum(v);
    if ((tid & 63) == 0) part[tid >> 6] = v;
    __syncthreads();
    double t = 0.0;
    if (tid == 0) {
        const int nw = (nthr + 63) >> 6;
        for (int w = 0; w < nw; ++w) t += part[w];
    }
    __syncthreads();
    return t;
}

__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_down(v, off, 64));
    return v;
}

// Minimum over a block (valid in thread 0); all threads must call it.
__device__ __forceinline__ double block_min(double v) {
    __shared__ double part[16];
    const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
    const int nthr = blockDim.x * blockDim.y * blockDim.z;
    v = wave_min(v);
    if ((tid & 63) == 0) part[tid >> 6] = v;
    __syncthreads();
    double t = v;
    if (tid == 0) {
        const int nw = (nthr + 63) >> 6;
        for (int w = 0; w < nw; ++w) t = fmin(t, part[w]);
    }
    __syncthreads();
    return t;
}

}  // namespace tph
