// FP64 vector kernels of the accelerators (Sec. "Accelerators").
//
// Flexible GMRES (Sec. "Comparison with FGMRES"): multi-vector dot products
// (with the vector's own norm in the same pass), fused axpy + norm
// (classical Gram-Schmidt with a second pass only on cancellation),
// normalisation and the solution update.  Flexible GCR (Alg. "Flexible
// GCR(m)"): one pass that finishes a step - orthogonalises and normalises
// the new direction pair (w, z) and updates x and r.  Anderson acceleration
// (Alg. "Anderson Acceleration(m) with Mixing"): dot products over the
// unknowns only and the mixing combination of the stored iterates.
//
// Residual-type vectors are flat (vx | vy | p) arrays whose entries outside
// the equation rows are zero, so those kernels are plain 1D streams.
// Reductions are two-stage with a fixed block count and fixed summation
// order: results are bitwise reproducible run to run (no atomics).
#include "kernels.h"
#include "reduce.h"

namespace tph {

int flat_blocks(size_t n) {
    size_t b = (n + 2047) / 2048;                     // >= 8 elements per thread
    if (b < 1) b = 1;
    if (b > 2048) b = 2048;
    return (int)b;
}

namespace {

constexpr int kNV = 8;
// two neighbouring entries (vectors are 256-byte aligned and of even length)
typedef double D2 __attribute__((ext_vector_type(2)));

// Partial sums of V_i . w for NV vectors per block, or one less: gridDim.y groups share the vectors evenly.  Index nv
// stands for w . w where norm_slot asks for it (of the entry of w that every thread has anyway).  How many vectors
// share a block does not change a sum (a block's threads, their strides and the tree over them
// are the same), only the work in flight: long vectors take up to 8 per block, so w is
// read once for them; short ones one each, so that every vector's loads and its
// reduction run side by side (up to 8 vectors of 25 500 entries: 4.4 us, against
// 11 us with all of them in each block and a barrier pair per vector).
// Bound by the reads of V (16 vectors of 3.35 M entries: 72 us, 6 TB/s).  LONG (more than 8 entries a thread): one
// load after the other, with all waves resident (1, 4, 8 and 16 vectors of 51 M entries: 128, 321, 575 and 1156 us; two
// entries' loads together 152, 355, 661 and 1285; eight slots in every block, those without a vector reading w again,
// 282, 382, 875 and 1514).  A kernel of its own: beside the other loop its scalar registers allow fewer waves than the
// 2048 blocks have (8 vectors: 885 us).
template <int NV, bool LONG>
__global__ __launch_bounds__(256) void k_multidot(const double* __restrict__ V0, size_t vstride, int nv,
                                                 const double* __restrict__ w, size_t n,
                                                 double* __restrict__ partial, int nblk, int norm_slot, Again again) {
    __shared__ double part[4 * (NV + 1)];
    if (again.asked() && !again.needed()) return;
    const int v0 = (int)(blockIdx.y * (unsigned)nv / gridDim.y), v1 = (int)((blockIdx.y + 1) * (unsigned)nv / gridDim.y);
    const double* V[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) V[v] = v0 + v < v1 ? V0 + (v0 + v) * vstride : w;
    double acc[NV + 1];
#pragma unroll
    for (int v = 0; v <= NV; ++v) acc[v] = 0.0;
    const size_t step = (size_t)gridDim.x * 256;
    size_t t = blockIdx.x * (size_t)256 + threadIdx.x;
    if constexpr (!LONG) {
        constexpr int U = NV >= 4 ? 2 : 8 / NV;      // entries in flight per thread
        for (; t + (U - 1) * step < n; t += U * step) {
            double x[U], y[U][NV];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                x[u] = w[t + u * step];
#pragma unroll
                for (int v = 0; v < NV; ++v) y[u][v] = V[v][t + u * step];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int v = 0; v < NV; ++v) acc[v] += y[u][v] * x[u];
                acc[NV] += x[u] * x[u];
            }
        }
    }
    for (; t < n; t += step) {
        const double x = w[t];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            acc[v] += V[v][t] * x;
            if (LONG) __builtin_amdgcn_sched_barrier(0);
        }
        acc[NV] += x * x;
    }
    const double s = block_sums(acc, part);
    const int v = threadIdx.x;
    if (v < v1 - v0) partial[(size_t)(v0 + v) * nblk + blockIdx.x] = s;
    if (v == NV && blockIdx.y == 0 && norm_slot >= 0) partial[(size_t)norm_slot * nblk + blockIdx.x] = s;
}

// Sums of U rows of at most kSumBlocks block sums (r, r + step, .. below k; valid in lane 0): a wave a row, the
// entries summed as by a workgroup with a thread for each.
constexpr int kSumBlocks = 128;
template <int U>
__device__ __forceinline__ void wave_row_sums(const double* __restrict__ partial, int nblk, int k, int r, int step,
                                              double (&t)[U]) {
    const int lane = threadIdx.x & 63;
    constexpr int Q = kSumBlocks / 64;
    double v[U][Q];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int b = q * 64 + lane;
            v[u][q] = b < nblk ? partial[(size_t)min(r + u * step, k - 1) * nblk + b] : 0.0;
        }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        t[u] = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) t[u] += wave_sum(0.0 + v[u][q]);
    }
}

// w -= sum_i h[i] V_i for any number of vectors, with the block sums of the new
// w . w, in one pass over w (8 vectors' loads in flight at a time; a launch per 8
// vectors re-read w and paid 5 us each on short vectors).  U entries a thread at once: 4 while its blocks
// leave the chip idle, 2 beyond 256 blocks, 1 where its strides over a long vector lie far apart (sums over 24
// steps: 290 k entries 452 us with 4, 481 with 2; 630 k 697, 673; 12.9 M entries and one vector 57 with 2, 47 with 1).
template <int U>
__global__ __launch_bounds__(256) void k_axpy_norm(double* __restrict__ w, const double* __restrict__ V0,
                                                  size_t vstride, int nv, const double* __restrict__ h, size_t n,
                                                  double* __restrict__ partial, Again again) {
    __shared__ double part[4];
    if (again.asked() && !again.needed()) return;
    double acc[1] = {0.0};
    const size_t step = (size_t)gridDim.x * 256;
    for (size_t t0 = blockIdx.x * (size_t)256 + threadIdx.x; t0 < n; t0 += U * step) {
        double x[U];
        bool in[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            in[u] = t0 + u * step < n;
            x[u] = in[u] ? w[t0 + u * step] : 0.0;
        }
        for (int v0 = 0; v0 < nv; v0 += kNV) {
            double y[U][kNV];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int v = 0; v < kNV; ++v)
                    y[u][v] = in[u] && v0 + v < nv ? V0[(v0 + v) * vstride + t0 + u * step] : 0.0;
#pragma unroll
            for (int v = 0; v < kNV; ++v) {
                const double hv = v0 + v < nv ? h[v0 + v] : 0.0;
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] -= hv * y[u][v];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!in[u]) continue;
            w[t0 + u * step] = x[u];
            acc[0] += x[u] * x[u];
        }
    }
    const double s = block_sums(acc, part);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// The same where h is not there yet, for vectors of at most kSumBlocks blocks (short ones: at most 8 entries a
// thread, byte offsets of 32 bits).  Every workgroup adds up the rows of block sums that h comes from by
// itself and the first one writes them out: that takes 1 us where a launch for it took 4.
// Bound by latency and by what a load costs to issue: vectors in uniform bases, a thread past the end
// reading the last entry (64-bit addresses and a mask per load took 8.8 us at 13 blocks and some 17 vectors, now 7.6).
__global__ __launch_bounds__(256) void k_axpy_norm_sums(double* __restrict__ w, const double* __restrict__ V0,
                                                       size_t vstride, int nv, unsigned n,
                                                       double* __restrict__ partial, RowSums rows, Again again) {
    __shared__ double part[4];
    __shared__ double hs[kMaxRestart + 2];
    if (again.asked() && !again.needed()) return;
    constexpr int RU = 4;                                // rows in flight per wave
    for (int r = threadIdx.x >> 6; r < rows.k; r += 4 * RU) {
        double t[RU];
        wave_row_sums<RU>(rows.partial, rows.nblk, rows.k, r, 4, t);
#pragma unroll
        for (int u = 0; u < RU; ++u)
            if ((threadIdx.x & 63) == 0 && r + 4 * u < rows.k) hs[r + 4 * u] = t[u];
    }
    __syncthreads();
    if (blockIdx.x == 0 && (int)threadIdx.x < rows.k) {
        rows.out[threadIdx.x] = hs[threadIdx.x];
        rows.host[threadIdx.x] = hs[threadIdx.x];
    }
    double acc[1] = {0.0};
    const unsigned step = gridDim.x * 256;
    constexpr int U = 4;
    auto entry = [](const double* base, unsigned byte) -> const double& { return *(const double*)((const char*)base + byte); };
    for (unsigned t0 = blockIdx.x * 256 + threadIdx.x; t0 < n; t0 += U * step) {
        double x[U];
        unsigned at[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            at[u] = min(t0 + u * step, n - 1) * 8u;
            x[u] = entry(w, at[u]);
        }
        int v0 = 0;
        for (; v0 + kNV <= nv; v0 += kNV) {
            double y[U][kNV];
#pragma unroll
            for (int v = 0; v < kNV; ++v)
#pragma unroll
                for (int u = 0; u < U; ++u) y[u][v] = entry(V0 + (v0 + v) * vstride, at[u]);
#pragma unroll
            for (int v = 0; v < kNV; ++v) {
                const double hv = hs[v0 + v];
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] -= hv * y[u][v];
            }
        }
        for (; v0 + 2 <= nv; v0 += 2) {
            double y[U][2];
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int u = 0; u < U; ++u) y[u][v] = entry(V0 + (v0 + v) * vstride, at[u]);
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const double hv = hs[v0 + v];
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] -= hv * y[u][v];
            }
        }
        if (v0 < nv) {
            const double hv = hs[v0];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] -= hv * entry(V0 + v0 * vstride, at[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (t0 + u * step >= n) continue;
            w[t0 + u * step] = x[u];
            acc[0] += x[u] * x[u];
        }
    }
    const double s = block_sums(acc, part);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// Row sums of partial (k rows of nblk) in one workgroup: 256 threads per row,
// four rows at a time, each in the same fixed order; rows of up to 128 entries by a
// wave each, which sums in that order too (20 rows of 44: 6.3 -> 5.3 us).  The results go to out and,
// where given, to mapped host memory, followed by the sequence number the host
// polls (one launch where a workgroup per row needed a second one to post it).
constexpr int kRowThreads = 256;
constexpr int kRowGroups = 4;
__global__ __launch_bounds__(kRowThreads * kRowGroups) void k_reduce_rows(
    const double* __restrict__ partial, int nblk, int k, double* __restrict__ out, double* __restrict__ host_out,
    unsigned* __restrict__ host_seq, unsigned seq, Again again) {
    __shared__ double part[kRowGroups][kRowThreads / 64];
    const int grp = threadIdx.x / kRowThreads, tid = threadIdx.x % kRowThreads;
    const bool left_out = again.asked() && !again.needed();
    if (nblk <= kSumBlocks) {                     // short rows: sixteen at a time, a wave each
        constexpr int U = 2, W = kRowThreads * kRowGroups / 64;
        for (int r = threadIdx.x >> 6; r < k; r += W * U) {
            double t[U];
            wave_row_sums<U>(partial, nblk, k, r, W, t);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (left_out) t[u] = *again.norm2;       // the norm that stays
                if ((threadIdx.x & 63) == 0 && r + u * W < k) {
                    out[r + u * W] = t[u];
                    if (host_out) host_out[r + u * W] = t[u];
                }
            }
        }
        k = 0;
    }
    for (int r0 = 0; r0 < k; r0 += kRowGroups) {
        const int r = r0 + grp;
        double s = 0.0;
        if (r < k) {
            const double* row = partial + (size_t)r * nblk;
            constexpr int U = 8;
            for (int b = tid; b < nblk; b += U * kRowThreads) {
                double a[U];
#pragma unroll
                for (int u = 0; u < U; ++u) a[u] = b + u * kRowThreads < nblk ? row[b + u * kRowThreads] : 0.0;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (b + u * kRowThreads < nblk) s += a[u];
            }
        }
        s = wave_sum(s);
        if ((tid & 63) == 0) part[grp][tid >> 6] = s;
        __syncthreads();
        if (tid == 0 && r < k) {
            double t = 0.0;
            for (int q = 0; q < kRowThreads / 64; ++q) t += part[grp][q];
            if (left_out) t = *again.norm2;       // the norm that stays
            out[r] = t;
            if (host_out) host_out[r] = t;
        }
        __syncthreads();
    }
    if (host_seq) {
        __threadfence_system();                   // every thread's values reach host memory first
        __syncthreads();
        if (threadIdx.x == 0) *(volatile unsigned*)host_seq = seq;
    }
}

__global__ __launch_bounds__(256) void k_scale_rnorm(double* __restrict__ dst, const double* __restrict__ src,
                                                    size_t n, const double* __restrict__ nrm2, Again again) {
    if (again.asked() && again.needed()) return;      // not the last pass
    const double r = 1.0 / sqrt(nrm2[0]);
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x)
        dst[t] = src[t] * r;
}

// x += sum_i y[i] Z_i, the coefficients in the kernel arguments
struct UpdateArgs {
    double* x;
    const double* Z0;
    size_t stride, n;
    int k;
    double y[kMaxRestart];
};
__global__ __launch_bounds__(256) void k_update_x(const UpdateArgs a) {
    for (size_t t = 2 * (blockIdx.x * (size_t)256 + threadIdx.x); t < a.n; t += (size_t)512 * gridDim.x) {
        D2 x = *(const D2*)(a.x + t);
        for (int v0 = 0; v0 < a.k; v0 += kNV) {
            D2 z[kNV];
#pragma unroll
            for (int v = 0; v < kNV; ++v)
                z[v] = v0 + v < a.k ? *(const D2*)(a.Z0 + (v0 + v) * a.stride + t) : D2{0.0, 0.0};
#pragma unroll
            for (int v = 0; v < kNV; ++v) x += (v0 + v < a.k ? a.y[v0 + v] : 0.0) * z[v];
        }
        *(D2*)(a.x + t) = x;
    }
}

// One step of flexible GCR after the Gram-Schmidt coefficients are known:
//   w^ = (w - sum_j hw_j W_j) / nu   (orth_w = 0: w is already orthogonal)
//   r -= alpha w^
// and, when z is given, z' = (z - sum_j hz_j Z_j) / nu, x += alpha z'.
// The coefficients travel in the kernel arguments (uniform scalar loads).
// One entry a thread: with 2048 blocks that stride over the vectors, long ones took 7 to 10 % more (51 M entries,
// 24 steps: 31.2 ms, now 28.1; two entries a thread 29.1, and 33.1 with 2048 blocks; 3.3 M entries 1.75, now 1.66).
__global__ __launch_bounds__(256) void k_gcr_step(const GcrStepArgs a) {
    const size_t t = blockIdx.x * (size_t)256 + threadIdx.x;
    if (t >= a.n) return;
    double wv = a.w[t];
    if (a.orth_w) {
#pragma unroll 4
        for (int j = 0; j < a.i; ++j) wv -= a.hw[j] * a.W0[j * a.stride + t];
    }
    wv *= a.inv_nu;
    a.w[t] = wv;
    a.r[t] -= a.alpha * wv;
    if (a.z) {
        double zv = a.z[t];
#pragma unroll 4
        for (int j = 0; j < a.i; ++j) zv -= a.hz[j] * a.Z0[j * a.stride + t];
        zv *= a.inv_nu;
        a.z[t] = zv;
        a.x[t] += a.alpha * zv;
    }
}

// Dot products of f with up to kNV vectors (and f . f) over the unknowns of a
// three-field solution vector only: vx rows 1..ny, columns 1..nx-1; vy rows
// 1..ny-1, columns 1..nx; p rows 1..ny, columns 1..nx.  Ghost entries (which
// repeat wall-adjacent values) and walls are left out.  Blocks stride over
// the 3 (ny + 2) rows, threads over the columns of a row.
__global__ __launch_bounds__(256) void k_multidot_unknowns(Geom g, size_t fstride, VecSet vs, int nv,
                                                          const double* __restrict__ f,
                                                          double* __restrict__ partial, int nblk, int norm_slot) {
    double acc[kNV];
#pragma unroll
    for (int v = 0; v < kNV; ++v) acc[v] = 0.0;
    double nacc = 0.0;
    const int rows = g.ny + 2;
    for (int q = blockIdx.x; q < 3 * rows; q += gridDim.x) {
        const int fld = q / rows, i = q - fld * rows;
        const int ilast = fld == 1 ? g.ny - 1 : g.ny;
        const int jlast = fld == 0 ? g.nx - 1 : g.nx;
        if (i < 1 || i > ilast) continue;
        const size_t row = (size_t)(kAlign - 1) + fld * fstride + (size_t)i * g.pitch;
        for (int j = 1 + threadIdx.x; j <= jlast; j += blockDim.x) {
            const double fv = f[row + j];
#pragma unroll
            for (int v = 0; v < kNV; ++v)
                if (v < nv) acc[v] += vs.v[v][row + j] * fv;
            nacc += fv * fv;
        }
    }
#pragma unroll
    for (int v = 0; v < kNV; ++v) {
        if (v < nv) {
            const double s = block_sum(acc[v]);
            if (threadIdx.x == 0) partial[(size_t)v * nblk + blockIdx.x] = s;
        }
    }
    if (norm_slot >= 0) {
        const double s = block_sum(nacc);
        if (threadIdx.x == 0) partial[(size_t)norm_slot * nblk + blockIdx.x] = s;
    }
}

// out = (acc ? out : 0) + sum_v (cx_v X_v + cf_v F_v) over every entry.  out
// may be one of the X_v: each entry is read before it is written, by the
// same thread.
__global__ __launch_bounds__(256) void k_mix(const MixArgs a) {
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < a.n; t += (size_t)gridDim.x * blockDim.x) {
        double s = a.acc ? a.out[t] : 0.0;
#pragma unroll
        for (int v = 0; v < kNV; ++v)
            if (v < a.nv) s += a.cx[v] * a.X[v][t] + a.cf[v] * a.F[v][t];
        a.out[t] = s;
    }
}

// posts seq to mapped host memory once every earlier kernel on the stream is done
__global__ void k_post_seq(unsigned* __restrict__ host_seq, unsigned seq) {
    __threadfence_system();
    *(volatile unsigned*)host_seq = seq;
}

__global__ __launch_bounds__(256) void k_p_sum(Geom g, const double* __restrict__ p, double* __restrict__ partial) {
    const int j = blockIdx.x * 64 + threadIdx.x + 1;
    const int i = blockIdx.y * 4 + threadIdx.y + 1;
    double v = 0.0;
    if (i <= g.ny && j <= g.nx) v = p[i * g.pitch + j];
    const double s = block_sum(v);
    if (threadIdx.x == 0 && threadIdx.y == 0) partial[blockIdx.y * gridDim.x + blockIdx.x] = s;
}

__global__ __launch_bounds__(256) void k_p_shift(Geom g, double* __restrict__ p, const double* __restrict__ sum) {
    const int j = blockIdx.x * 64 + threadIdx.x + 1;
    const int i = blockIdx.y * 4 + threadIdx.y + 1;
    if (i > g.ny || j > g.nx) return;
    p[i * g.pitch + j] -= sum[0] / ((double)g.nx * (double)g.ny);
}

}  // namespace

hipError_t launch_multidot(const double* V0, size_t vstride, int nv, const double* w, size_t n, double* partial,
                           int nblk, hipStream_t st, int norm_slot, Again again) {
    // vectors per block: up to 8 once the blocks of one group fill the chip by
    // themselves (two per CU), fewer while they do not; nblk is n / 2048
    const int per = nblk >= 512 ? 8 : nblk >= 128 ? 4 : 1;
    const int groups = (nv + per - 1) / per;
    if (groups < 1) return hipErrorInvalidValue;
    const dim3 grid(nblk, groups);
    const bool lng = n > (size_t)2048 * nblk;        // the block count is at its most
#define TPH_DOT(NV)                                                                                                    \
    case NV:                                                                                                           \
        if (lng)                                                                                                       \
            hipLaunchKernelGGL((k_multidot<NV, true>), grid, dim3(256), 0, st, V0, vstride, nv, w, n, partial, nblk,   \
                               norm_slot, again);                                                                      \
        else                                                                                                           \
            hipLaunchKernelGGL((k_multidot<NV, false>), grid, dim3(256), 0, st, V0, vstride, nv, w, n, partial, nblk,  \
                               norm_slot, again);                                                                      \
        break;
    switch ((nv + groups - 1) / groups) {            // the largest group's
        TPH_DOT(1)
        TPH_DOT(2)
        TPH_DOT(3)
        TPH_DOT(4)
        TPH_DOT(5)
        TPH_DOT(6)
        TPH_DOT(7)
        TPH_DOT(8)
    }
#undef TPH_DOT
    return hipGetLastError();
}

hipError_t launch_axpy_norm(double* w, const double* V0, size_t vstride, int nv, const double* h, size_t n,
                            double* partial, int nblk, hipStream_t st, Again again) {
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nblk), dim3(256), 0, st, w, V0, vstride, nv, h, n, partial, again);
    };
    if (n > (size_t)2048 * nblk) launch(k_axpy_norm<1>);
    else if (nblk > 256) launch(k_axpy_norm<2>);
    else launch(k_axpy_norm<4>);
    return hipGetLastError();
}

int sum_blocks_max() { return kSumBlocks; }

hipError_t launch_axpy_norm_sums(double* w, const double* V0, size_t vstride, int nv, const RowSums& rows, size_t n,
                                 double* partial, hipStream_t st, Again again) {
    if (rows.nblk < 1 || rows.nblk > kSumBlocks || n < 1 || n > (size_t)kSumBlocks * 2048 || rows.k < nv || rows.k < 1 || rows.k > kMaxRestart + 2)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_axpy_norm_sums, dim3(rows.nblk), dim3(256), 0, st, w, V0, vstride, nv, (unsigned)n, partial, rows,
                       again);
    return hipGetLastError();
}

hipError_t launch_reduce_rows(const double* partial, int nblk, int k, double* out, hipStream_t st,
                              double* host_out, unsigned* host_seq, unsigned seq, Again again) {
    hipLaunchKernelGGL(k_reduce_rows, dim3(1), dim3(kRowThreads * kRowGroups), 0, st, partial, nblk, k, out, host_out,
                       host_seq, seq, again);
    return hipGetLastError();
}

hipError_t launch_scale_by_rnorm(double* dst, const double* src, size_t n, const double* nrm2, hipStream_t st,
                                 Again again) {
    hipLaunchKernelGGL(k_scale_rnorm, dim3(flat_blocks(n)), dim3(256), 0, st, dst, src, n, nrm2, again);
    return hipGetLastError();
}

hipError_t launch_update_x(double* x, const double* Z0, size_t zstride, int k, const double* y, size_t n,
                           hipStream_t st) {
    if (k < 0 || k > kMaxRestart || (n & 1) || (zstride & 1)) return hipErrorInvalidValue;
    UpdateArgs a{};
    a.x = x;
    a.Z0 = Z0;
    a.stride = zstride;
    a.n = n;
    a.k = k;
    for (int v = 0; v < k; ++v) a.y[v] = y[v];
    const size_t b = (n + 511) / 512;
    hipLaunchKernelGGL(k_update_x, dim3((unsigned)(b < 1 ? 1 : b > 2048 ? 2048 : b)), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_gcr_step(const GcrStepArgs& a, hipStream_t st) {
    if (a.i < 0 || a.i > kMaxRestart || a.n < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_gcr_step, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, st, a);
    return hipGetLastError();
}

int unknown_dot_blocks(const Geom& g) {
    const int rows = 3 * (g.ny + 2);
    return rows < 2048 ? rows : 2048;
}

hipError_t launch_multidot_unknowns(const Geom& g, size_t fstride, const double* const* vecs, int nv,
                                    const double* f, double* partial, int nblk, hipStream_t st, int norm_slot) {
    if (nv == 0 && norm_slot >= 0) {
        VecSet vs{};
        hipLaunchKernelGGL(k_multidot_unknowns, dim3(nblk), dim3(256), 0, st, g, fstride, vs, 0, f, partial, nblk,
                           norm_slot);
        return hipGetLastError();
    }
    for (int v0 = 0; v0 < nv; v0 += kNV) {
        const int c = nv - v0 < kNV ? nv - v0 : kNV;
        VecSet vs{};
        for (int v = 0; v < c; ++v) vs.v[v] = vecs[v0 + v];
        const int ns = (v0 == 0 && norm_slot >= 0) ? norm_slot : -1;
        hipLaunchKernelGGL(k_multidot_unknowns, dim3(nblk), dim3(256), 0, st, g, fstride, vs, c, f,
                           partial + (size_t)v0 * nblk, nblk, ns);
    }
    return hipGetLastError();
}

hipError_t launch_mix(double* out, const double* const* X, const double* cx, const double* const* F,
                      const double* cf, int nv, size_t n, hipStream_t st) {
    for (int v0 = 0; v0 < nv; v0 += kNV) {
        MixArgs a{};
        a.out = out;
        a.n = n;
        a.nv = nv - v0 < kNV ? nv - v0 : kNV;
        a.acc = v0 > 0 ? 1 : 0;
        for (int v = 0; v < a.nv; ++v) {
            a.X[v] = X[v0 + v];
            a.F[v] = F[v0 + v];
            a.cx[v] = cx[v0 + v];
            a.cf[v] = cf[v0 + v];
        }
        hipLaunchKernelGGL(k_mix, dim3(flat_blocks(n)), dim3(256), 0, st, a);
    }
    return hipGetLastError();
}

hipError_t launch_post_seq(unsigned* host_seq, unsigned seq, hipStream_t st) {
    hipLaunchKernelGGL(k_post_seq, dim3(1), dim3(1), 0, st, host_seq, seq);
    return hipGetLastError();
}

hipError_t launch_p_sum(const Geom& g, const double* p, double* partial, int* nblk_out, hipStream_t st) {
    const dim3 grid((g.nx + 63) / 64, (g.ny + 3) / 4);
    if (nblk_out) *nblk_out = (int)(grid.x * grid.y);
    hipLaunchKernelGGL(k_p_sum, grid, dim3(64, 4), 0, st, g, p, partial);
    return hipGetLastError();
}

hipError_t launch_p_shift(const Geom& g, double* p, const double* sum, hipStream_t st) {
    const dim3 grid((g.nx + 63) / 64, (g.ny + 3) / 4);
    hipLaunchKernelGGL(k_p_shift, grid, dim3(64, 4), 0, st, g, p, sum);
    return hipGetLastError();
}

}  // namespace tph
