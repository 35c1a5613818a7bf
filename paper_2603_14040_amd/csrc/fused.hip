// Single-problem launchers of the fused multigrid kernels (device bodies in
// fused_dev.h): LDS-tiled smoothing sweep, fused residual + restriction,
// single-workgroup coarse tail.
#include <hip/hip_ext.h>

#include "fused_dev.h"
#include "tail_dev.h"

namespace tph {
namespace {

using namespace dev;

template <typename T, int TW, int TH, int SM, int MODE>
__global__ __launch_bounds__(kTileThreads, kTileWaves) void k_smooth_tile(Geom g, Geom gc, const T* __restrict__ exi,
                                                    const T* __restrict__ eyi, T* __restrict__ exo,
                                                    T* __restrict__ eyo, const T* __restrict__ rx,
                                                    const T* __restrict__ ry, const T* __restrict__ eb,
                                                    const T* __restrict__ ep, const T* __restrict__ ecx,
                                                    const T* __restrict__ ecy, T omega) {
    int tbx, tby;
    xcd_tile(tbx, tby);
    smooth_tile_body<T, TW, TH, SM, MODE>(g, gc, exi, eyi, exo, eyo, rx, ry, eb, ep, ecx, ecy, omega, tbx, tby);
}

template <typename T, int CTW, int CTH>
__global__ __launch_bounds__(CTW * CTH) void k_res_restrict(Geom g, Geom gc, const T* __restrict__ ex,
                                                           const T* __restrict__ ey, const T* __restrict__ rx,
                                                           const T* __restrict__ ry, const T* __restrict__ eb,
                                                           const T* __restrict__ ep, T* __restrict__ rcx,
                                                           T* __restrict__ rcy) {
    int tbx, tby;
    xcd_tile(tbx, tby);
    res_restrict_body<T, CTW, CTH>(g, gc, ex, ey, rx, ry, eb, ep, rcx, rcy, tbx, tby);
}

template <typename T, int NT, int KP>
__global__ __launch_bounds__(NT) void k_coarse_cycle(CoarseArgs<T> A) {
    coarse_cycle_body<T, NT, KP>(A);
}

template <typename T, int NT, int KP>
hipError_t launch_tail(const CoarseArgs<T>& a, size_t lds_bytes, hipStream_t st) {
    hipLaunchKernelGGL((k_coarse_cycle<T, NT, KP>), dim3(1), dim3(NT), lds_bytes, st, a);
    return hipGetLastError();
}

}  // namespace


template <typename T>
size_t coarse_cycle_lds_bytes(const Geom* g, int nl, int nc) {
    size_t n = dev::tail_area<T>(g[0].nx, g[0].ny) + 16;
    for (int l = 1; l < nl; ++l) n += (l < nl - 1 ? 3 : 1) * dev::tail_area<T>(g[l].nx, g[l].ny);
    return n + (size_t)dev::tail_dense_pad(nc) * sizeof(double);
}

// as few threads as own the top level's cell pairs one each (fewer waves meet
// at every barrier); two pairs per thread beyond 512, four beyond 1024
TailShape coarse_cycle_shape(int nx, int ny) {
    const int pairs = (nx / 2) * ny;
    if (pairs <= 256) return {256, 1};
    return {512, pairs <= 512 ? 1 : pairs <= 1024 ? 2 : 4};
}

template <typename T>
hipError_t launch_smooth_tile(const Geom& g, const Geom* gc, int smoother, int mode, const T* exi, const T* eyi,
                              T* exo, T* eyo, const T* rx, const T* ry, const T* eb, const T* ep, const T* ecx,
                              const T* ecy, T omega, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
    constexpr int TW = kTileW, TH = tile_h<T>();
    const dim3 grid((g.nx + TW - 1) / TW, (g.ny + TH - 1) / TH);
    const Geom gcc = gc ? *gc : g;
#define TPH_SMT(SM, MODE)                                                                                        \
    do {                                                                                                          \
        if (t0)                                                                                                   \
            hipExtLaunchKernelGGL((k_smooth_tile<T, TW, TH, SM, MODE>), grid, dim3(kTileThreads), 0, st, t0, t1, \
                                  0, g, gcc, exi, eyi, exo, eyo, rx, ry, eb, ep, ecx, ecy, omega);              \
        else                                                                                                      \
            hipLaunchKernelGGL((k_smooth_tile<T, TW, TH, SM, MODE>), grid, dim3(kTileThreads), 0, st, g, gcc, exi, \
                               eyi, exo, eyo, rx, ry, eb, ep, ecx, ecy, omega);                                   \
    } while (0)
    if (smoother == kSmGS) {
        if (mode == kModeZero) TPH_SMT(kSmGS, kModeZero);
        else if (mode == kModeProlong) TPH_SMT(kSmGS, kModeProlong);
        else TPH_SMT(kSmGS, kModePlain);
    } else {
        if (mode == kModeZero) TPH_SMT(kSmJacobi, kModeZero);
        else if (mode == kModeProlong) TPH_SMT(kSmJacobi, kModeProlong);
        else TPH_SMT(kSmJacobi, kModePlain);
    }
#undef TPH_SMT
    return hipGetLastError();
}

template <typename T>
hipError_t launch_res_restrict(const Geom& gf, const Geom& gc, const T* ex, const T* ey, const T* rx, const T* ry,
                               const T* eb, const T* ep, T* rcx, T* rcy, hipStream_t st) {
    constexpr int CTW = kRRTileW, CTH = rr_tile_h<T>();
    const dim3 grid((gc.nx + CTW - 1) / CTW, (gc.ny + CTH - 1) / CTH);
    hipLaunchKernelGGL((k_res_restrict<T, CTW, CTH>), grid, dim3(CTW * CTH), 0, st, gf, gc, ex, ey, rx, ry, eb, ep,
                       rcx, rcy);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_coarse_cycle(const CoarseArgs<T>& a, size_t lds_bytes, hipStream_t st) {
    const TailShape sh = coarse_cycle_shape(a.lv[0].nx, a.lv[0].ny);
    if ((a.lv[0].nx / 2) * a.lv[0].ny > sh.threads * sh.pairs || lds_bytes > kTailLdsMax) return hipErrorInvalidValue;
    if (sh.threads == 256) return launch_tail<T, 256, 1>(a, lds_bytes, st);
    if (sh.pairs == 1) return launch_tail<T, 512, 1>(a, lds_bytes, st);
    if (sh.pairs == 2) return launch_tail<T, 512, 2>(a, lds_bytes, st);
    // a FP64 tail of more than 2048 cells does not fit the LDS
    if constexpr (sizeof(T) == 4) return launch_tail<T, 512, 4>(a, lds_bytes, st);
    else return hipErrorInvalidValue;
}

#define TPH_INST(T)                                                                                                \
    template size_t coarse_cycle_lds_bytes<T>(const Geom*, int, int);                                             \
    template hipError_t launch_smooth_tile<T>(const Geom&, const Geom*, int, int, const T*, const T*, T*, T*,       \
                                              const T*, const T*, const T*, const T*, const T*, const T*, T,         \
                                              hipStream_t, hipEvent_t, hipEvent_t);                                 \
    template hipError_t launch_res_restrict<T>(const Geom&, const Geom&, const T*, const T*, const T*, const T*,    \
                                               const T*, const T*, T*, T*, hipStream_t);                            \
    template hipError_t launch_coarse_cycle<T>(const CoarseArgs<T>&, size_t, hipStream_t);
TPH_INST(float)
TPH_INST(double)
#undef TPH_INST

}  // namespace tph
