// Coarsest-level solve in FP64 (Ch. 4 "Multigrid Cycles": the coarsest
// correction equation is solved directly).  The dense matrix M = -L of the
// coarsest level (symmetric positive definite) is assembled on the device
// from the rediscretised stencil, inverted once per coefficient set by an
// in-place Gauss-Jordan elimination (a single problem's in panels of 32 steps
// over the device, a batch's small ones by one workgroup each), and applied as a
// dense matrix-vector product (one wavefront per row).  Unknown order: vx(i, j)
// row-major (i in [1, ny], j in [1, nx-1]), then vy(i, j) (i in [1, ny-1],
// j in [1, nx]).
#include "kernels.h"
#include "reduce.h"

namespace tph {

int coarse_unknowns(const Geom& g) { return g.ny * (g.nx - 1) + (g.ny - 1) * g.nx; }

namespace {

__device__ __forceinline__ void unknown_to_node(const Geom& g, int m, int& comp, int& i, int& j) {
    const int nvx = g.ny * (g.nx - 1);
    if (m < nvx) {
        comp = 0;
        i = 1 + m / (g.nx - 1);
        j = 1 + m % (g.nx - 1);
    } else {
        m -= nvx;
        comp = 1;
        i = 1 + m / g.nx;
        j = 1 + m % g.nx;
    }
}

// Column of coef * field(ci, cj) in a row of M = -L, walls dropped (-1) and ghosts mirrored onto the
// adjacent unknown (coef with them).
__device__ __forceinline__ int column_of(const Geom& g, int comp, int ci, int cj, double& coef) {
    const int nvx = g.ny * (g.nx - 1);
    if (comp == 0) {
        if (cj <= 0 || cj >= g.nx) return -1;
        if (ci == 0) { ci = 1; coef *= g.mir[2]; }
        else if (ci == g.ny + 1) { ci = g.ny; coef *= g.mir[3]; }
        return (ci - 1) * (g.nx - 1) + (cj - 1);
    }
    if (ci <= 0 || ci >= g.ny) return -1;
    if (cj == 0) { cj = 1; coef *= g.mir[0]; }
    else if (cj == g.nx + 1) { cj = g.nx; coef *= g.mir[1]; }
    return nvx + (ci - 1) * g.nx + (cj - 1);
}

// One workgroup per row: every lane knows the row's nine entries and writes the columns it comes to,
// zeros and sums (a mirrored ghost meets an entry of its own), once and in whole lines.  A thread per row
// that cleared it and added the entries in memory took 15 us at 112 unknowns and 49 us at 420.
__global__ __launch_bounds__(64) void k_coarse_assemble(Geom g, const double* __restrict__ eb,
                                                        const double* __restrict__ ep, double* __restrict__ M, int n) {
    const int m = blockIdx.x;
    int comp, i, j;
    unknown_to_node(g, m, comp, i, j);
    const int P = g.pitch;
    const int c = i * P + j;
    const double idx2 = g.idx2, idy2 = g.idy2, idxy = 1.0 / (g.dx * g.dy);
    int at[9];
    double v[9];
    int k = 0;
    auto add = [&](int cp, int ci, int cj, double coef) {
        at[k] = column_of(g, cp, ci, cj, coef);
        v[k++] = coef;
    };
    if (comp == 0) {
        const double er = ep[c + 1], el = ep[c], bt = eb[c], bb = eb[c - P];
        add(0, i, j + 1, 2 * er * idx2);
        add(0, i, j, -2 * (er + el) * idx2 - (bt + bb) * idy2);
        add(0, i, j - 1, 2 * el * idx2);
        add(0, i + 1, j, bt * idy2);
        add(0, i - 1, j, bb * idy2);
        add(1, i, j + 1, bt * idxy);
        add(1, i, j, -bt * idxy);
        add(1, i - 1, j + 1, -bb * idxy);
        add(1, i - 1, j, bb * idxy);
    } else {
        const double et = ep[c + P], eb_ = ep[c], br = eb[c], bl = eb[c - 1];
        add(1, i + 1, j, 2 * et * idy2);
        add(1, i, j, -2 * (et + eb_) * idy2 - (br + bl) * idx2);
        add(1, i - 1, j, 2 * eb_ * idy2);
        add(1, i, j + 1, br * idx2);
        add(1, i, j - 1, bl * idx2);
        add(0, i + 1, j, br * idxy);
        add(0, i, j, -br * idxy);
        add(0, i + 1, j - 1, -bl * idxy);
        add(0, i, j - 1, bl * idxy);
    }
    double* row = M + (size_t)m * n;
    for (int q = threadIdx.x; q < n; q += 64) {
        double sum = 0.0;
#pragma unroll
        for (int t = 0; t < 9; ++t) sum = at[t] == q ? sum - v[t] : sum;
        row[q] = sum;
    }
}

// In-place Gauss-Jordan inverse of an SPD matrix (no pivoting needed), kPanel steps per pair of launches.
// Step k scales row k by 1 / M[k][k] and takes M[i][k] times it from every other row; an entry (i, j) needs
// of a step only f = M[i][k] and p = M[k][j] / M[k][k] as they are then.
//   k_gj_panel:  these factors for the panel's steps, F[s][i] and P[s][j].  A workgroup takes the panel's
//                rows and columns and 32 further rows (for F) or columns (for P), and steps through those
//                alone: entries in registers, row and column s published through LDS, one barrier a step.
//   k_gj_update: every entry of a 32 x 32 tile through all the steps, the factors in LDS.
// Each entry sees the operations of the plain algorithm in the same order.  Bound by the chain of n
// pivots, about 0.5 us each (publish, barrier, division, update); a pair of launches per pivot took 4.8 us.
// n = 212: 1030 us, now 213; n = 112: 278 us by one workgroup, now 114.
constexpr int kPanel = 32;

// SIDE 0: rows [k0, k0 + 32) and [t0, t0 + 32) of the panel's columns; 1: the transpose
template <int SIDE>
__device__ __forceinline__ void gj_panel(const double* __restrict__ M, int n, int k0, int t0,
                                         double* __restrict__ out, double (*prow)[2 * kPanel],
                                         double (*pcol)[2 * kPanel], double (*kept)[kPanel]) {
    constexpr int NC = SIDE == 0 ? kPanel / 4 : 2 * kPanel / 4;        // threads across: 4 columns each, 2 rows
    const int r0 = (threadIdx.x / NC) * 2, c0 = (threadIdx.x % NC) * 4;
    // position relative to the panel: 0 .. 31 within, others are further rows or columns (or the panel's own again)
    int gr[2], gc[4];
#pragma unroll
    for (int r = 0; r < 2; ++r) gr[r] = r0 + r < kPanel ? r0 + r : t0 + r0 + r - kPanel - k0;
#pragma unroll
    for (int c = 0; c < 4; ++c) gc[c] = c0 + c < kPanel ? c0 + c : t0 + c0 + c - kPanel - k0;
    double a[2][4];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int i = k0 + gr[r], j = k0 + gc[c];
            a[r][c] = i < n && j < n ? M[(size_t)i * n + j] : 0.0;
        }
    const int steps = min(kPanel, n - k0);
    for (int s4 = 0; s4 < steps; s4 += 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int s = s4 + q;
            if (s >= steps) break;                                     // the same for every thread
            double* pr = prow[q & 1];                                  // two buffers: one barrier a step
            double* pc = pcol[q & 1];
            if (r0 == s4 + (q & 2)) {
#pragma unroll
                for (int c = 0; c < 4; ++c) pr[c0 + c] = a[q & 1][c];
            }
            if (c0 == s4) {
#pragma unroll
                for (int r = 0; r < 2; ++r) pc[r0 + r] = a[r][q];
            }
            __syncthreads();
            const double rd = 1.0 / pr[s];
            double p[4], f[2];
#pragma unroll
            for (int c = 0; c < 4; ++c) p[c] = gc[c] == s ? rd : pr[c0 + c] * rd;
#pragma unroll
            for (int r = 0; r < 2; ++r) f[r] = pc[r0 + r];
            // kept until the end: the barrier would wait for a store to memory
            if (SIDE == 0) {
                if (c0 == 0 && r0 >= kPanel) {
#pragma unroll
                    for (int r = 0; r < 2; ++r) kept[s][r0 + r - kPanel] = f[r];
                }
            } else if (r0 == 0 && c0 >= kPanel) {
#pragma unroll
                for (int c = 0; c < 4; ++c) kept[s][c0 + c - kPanel] = p[c];
            }
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    a[r][c] = gr[r] == s ? p[c] : gc[c] == s ? -f[r] * rd : __builtin_fma(-f[r], p[c], a[r][c]);
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < steps * kPanel; t += 256)
        if (t0 + t % kPanel < n) out[(size_t)(t / kPanel) * n + t0 + t % kPanel] = kept[t / kPanel][t % kPanel];
}

__global__ __launch_bounds__(256) void k_gj_panel(const double* __restrict__ M, int n, int k0,
                                                  double* __restrict__ F, double* __restrict__ P) {
    __shared__ double prow[2][2 * kPanel], pcol[2][2 * kPanel], kept[kPanel][kPanel];
    const int t0 = (int)blockIdx.x * kPanel;
    if (blockIdx.y == 0) gj_panel<0>(M, n, k0, t0, F, prow, pcol, kept);
    else gj_panel<1>(M, n, k0, t0, P, prow, pcol, kept);
}

__global__ __launch_bounds__(256) void k_gj_update(double* __restrict__ M, int n, int k0, const double* __restrict__ F,
                                                   const double* __restrict__ P) {
    __shared__ double f[kPanel][kPanel], p[kPanel][kPanel];
    const int i0 = (int)blockIdx.y * kPanel, j0 = (int)blockIdx.x * kPanel;
    const int steps = min(kPanel, n - k0);
    for (int t = threadIdx.x; t < kPanel * kPanel; t += 256) {         // steps past the last: factors of zero, no change
        const int s = t / kPanel, l = t % kPanel;
        f[s][l] = s < steps && i0 + l < n ? F[(size_t)s * n + i0 + l] : 0.0;
        p[s][l] = s < steps && j0 + l < n ? P[(size_t)s * n + j0 + l] : 0.0;
    }
    const int l = threadIdx.x % kPanel, r0 = threadIdx.x / kPanel;     // column, first of the rows r0 + 8 q
    const int j = j0 + l;
    double a[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = i0 + r0 + 8 * q < n && j < n ? M[(size_t)(i0 + r0 + 8 * q) * n + j] : 0.0;
    __syncthreads();
    if (i0 != k0 && j0 != k0) {                                        // k0 is a multiple of the tile's size
#pragma unroll 8
        for (int s = 0; s < kPanel; ++s) {
#pragma unroll
            for (int q = 0; q < 4; ++q) a[q] = __builtin_fma(-f[s][r0 + 8 * q], p[s][l], a[q]);
        }
    } else {
#pragma unroll 4
        for (int s = 0; s < kPanel; ++s) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double fs = f[s][r0 + 8 * q], ps = p[s][l];
                a[q] = i0 + r0 + 8 * q == k0 + s ? ps : j == k0 + s ? -fs * ps : __builtin_fma(-fs, ps, a[q]);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (i0 + r0 + 8 * q < n && j < n) M[(size_t)(i0 + r0 + 8 * q) * n + j] = a[q];
}

// Gauss-Jordan inversion of a small SPD matrix (n <= kGJLds) by one
// workgroup of kGJThreads threads, the matrix held in registers: R =
// kGJThreads / n threads share a row, each owning a run of at most kGJRun
// consecutive entries.  Each step k copies the old row k and column k to
// LDS, then every thread updates its own entries (the same operations as
// the device-wide form: row k scaled by 1 / M[k][k], the others reduced by
// the scaled row), two barriers per step.  Blocks each invert their own
// matrix (mats[blockIdx.x], sizes ns[blockIdx.x]): one launch for a batch, 278 us
// at n = 112 however many there are up to the number of CUs.
constexpr int kGJThreads = 1024;
constexpr int kGJRun = 20;   // max over n <= 136 of ceil(n / floor(1024 / n))
static_assert(kGJThreads >= kGJLds, "one row per thread at least");

__global__ __launch_bounds__(kGJThreads) void k_gauss_jordan_lds(double* const* __restrict__ mats,
                                                                const int* __restrict__ ns) {
    extern __shared__ double lds[];
    const int n = ns[blockIdx.x];
    double* __restrict__ Mg = mats[blockIdx.x];
    double* prow = lds;
    double* pcol = lds + n;
    const int tid = threadIdx.x;
    const int R = kGJThreads / n;                   // threads per row
    const int ch = (n + R - 1) / R;                 // run length
    const int i = tid / R, p = tid - (tid / R) * R;
    const int j0 = p * ch;
    const int cnt = i < n ? (j0 + ch <= n ? ch : (j0 < n ? n - j0 : 0)) : 0;
    double a[kGJRun];
#pragma unroll
    for (int c = 0; c < kGJRun; ++c) a[c] = c < cnt ? Mg[(size_t)i * n + j0 + c] : 0.0;
    for (int k = 0; k < n; ++k) {
#pragma unroll
        for (int c = 0; c < kGJRun; ++c) {
            if (c < cnt) {
                if (i == k) prow[j0 + c] = a[c];
                if (j0 + c == k) pcol[i] = a[c];
            }
        }
        __syncthreads();
        const double rd = 1.0 / pcol[k];
        const double f = cnt > 0 ? pcol[i] : 0.0;
#pragma unroll
        for (int c = 0; c < kGJRun; ++c) {
            if (c < cnt) {
                const int j = j0 + c;
                if (i == k) a[c] = j == k ? rd : a[c] * rd;
                else a[c] = j == k ? -f * rd : a[c] - f * (prow[j] * rd);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int c = 0; c < kGJRun; ++c)
        if (c < cnt) Mg[(size_t)i * n + j0 + c] = a[c];
}

template <typename T>
__global__ __launch_bounds__(256) void k_coarse_solve(Geom g, const double* __restrict__ Minv,
                                                      const T* __restrict__ rx, const T* __restrict__ ry,
                                                      T* __restrict__ ex, T* __restrict__ ey, int n) {
    extern __shared__ double rs[];
    const int tid = threadIdx.x;
    const int P = g.pitch;
    for (int m = tid; m < n; m += blockDim.x) {
        int comp, i, j;
        unknown_to_node(g, m, comp, i, j);
        rs[m] = (double)(comp == 0 ? rx[i * P + j] : ry[i * P + j]);
    }
    __syncthreads();
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int nwave = blockDim.x >> 6;
    // one wave per row of the inverse; every workgroup holds the whole right-hand side
    for (int m = blockIdx.x * nwave + wave; m < n; m += gridDim.x * nwave) {
        const double* row = Minv + (size_t)m * n;
        double s = 0.0;
        for (int q = lane; q < n; q += 64) s += row[q] * rs[q];
        s = wave_sum(s);
        if (lane == 0) {
            // L e = r  <=>  e = -(-L)^{-1} r
            const T e = (T)(-s);
            int comp, i, j;
            unknown_to_node(g, m, comp, i, j);
            const int c = i * P + j;
            if (comp == 0) {
                ex[c] = e;
                if (i == 1) ex[c - P] = (T)g.mir[2] * e;
                if (i == g.ny) ex[c + P] = (T)g.mir[3] * e;
            } else {
                ey[c] = e;
                if (j == 1) ey[c - 1] = (T)g.mir[0] * e;
                if (j == g.nx) ey[c + 1] = (T)g.mir[1] * e;
            }
        }
    }
}

}  // namespace

hipError_t launch_coarse_assemble(const Geom& g, const double* eb, const double* ep, double* M, hipStream_t st) {
    const int n = coarse_unknowns(g);
    hipLaunchKernelGGL(k_coarse_assemble, dim3(n), dim3(64), 0, st, g, eb, ep, M, n);
    return hipGetLastError();
}

size_t gauss_jordan_lds_bytes(int n) { return 2 * (size_t)n * sizeof(double); }

hipError_t launch_gauss_jordan_batched(double* const* mats, const int* ns, int count, int nmax, hipStream_t st) {
    const size_t lds = gauss_jordan_lds_bytes(nmax);
    if (nmax > kGJLds) return hipErrorInvalidValue;
    static thread_local int dev_cached = -1;
    static thread_local size_t granted = 64 * 1024;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return hipGetLastError();
    if (dev != dev_cached) {
        dev_cached = dev;
        granted = 64 * 1024;
    }
    if (lds > granted) {
        const hipError_t e = hipFuncSetAttribute((const void*)k_gauss_jordan_lds,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return e;
        }
        granted = lds;
    }
    hipLaunchKernelGGL(k_gauss_jordan_lds, dim3(count), dim3(kGJThreads), lds, st, mats, ns);
    return hipGetLastError();
}

size_t gauss_jordan_work(int n) { return 2 * (size_t)kPanel * n; }

hipError_t launch_gauss_jordan(double* M, int n, hipStream_t st, double* work) {
    if (!work) return hipErrorInvalidValue;
    double* F = work;
    double* P = work + (size_t)kPanel * n;
    const unsigned tiles = (unsigned)((n + kPanel - 1) / kPanel);
    for (int k0 = 0; k0 < n; k0 += kPanel) {
        hipLaunchKernelGGL(k_gj_panel, dim3(tiles, 2), dim3(256), 0, st, M, n, k0, F, P);
        hipLaunchKernelGGL(k_gj_update, dim3(tiles, tiles), dim3(256), 0, st, M, n, k0, F, P);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_coarse_solve(const Geom& g, const double* Minv, const T* rx, const T* ry, T* ex, T* ey,
                               hipStream_t st) {
    const int n = coarse_unknowns(g);
    // 4 rows per workgroup: the n^2 inverse streams through the whole device
    hipLaunchKernelGGL(k_coarse_solve<T>, dim3((n + 3) / 4), dim3(256), (size_t)n * sizeof(double), st, g, Minv, rx,
                       ry, ex, ey, n);
    return hipGetLastError();
}

template hipError_t launch_coarse_solve<float>(const Geom&, const double*, const float*, const float*, float*,
                                               float*, hipStream_t);
template hipError_t launch_coarse_solve<double>(const Geom&, const double*, const double*, const double*,
                                                double*, double*, hipStream_t);

}  // namespace tph
