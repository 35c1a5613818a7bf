// Device bodies of the fused multigrid kernels, shared by the single-problem
// kernels (fused.hip) and the batched kernels (batch.hip).
//
// smooth_tile_body: one full smoothing sweep on an LDS tile.
//   Gauss-Seidel: the four colour half-sweeps (vx red, vx black, vy red,
//   vy black) run inside the tile; each half-sweep needs the result of the
//   previous one one node further out, so the tile loads a halo of 4 nodes
//   and updates shrinking regions (halo 3, 2, 1, 0).  The sweep reads the
//   old iterate from one buffer and writes the interior of the tile to the
//   other, so overlapping tiles never see each other's new values and the
//   result equals the four separate half-sweeps exactly.
//   Jacobi: one stage, halo 1.
//   Modes: plain, zero initial guess (no load of the iterate), and
//   prolongation + correction fused into the load (bilinear coarse-to-fine
//   interpolation from an LDS window of the coarse correction, ghosts
//   re-mirrored).
// res_restrict_body: residual r - L e on the fine footprint of a tile of
//   coarse cells, kept in LDS, then the normalised restriction (gather form
//   of Alg. "4-Color Parallel Restriction"); the fine residual never goes
//   to memory.
#pragma once
#include "kernels.h"
#include "reduce.h"
#include "stencil.h"

namespace tph {
namespace dev {


// a * b + c with one rounding, where which product of a sum of two goes inside
// must not depend on the code around it
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

enum { kModePlain = kTilePlain, kModeZero = kTileZero, kModeProlong = kTileProlong };
enum { kSmJacobi = 0, kSmGS = 1 };

__device__ __forceinline__ bool is_vx(const Geom& g, int i, int j) { return i >= 1 && i <= g.ny && j >= 1 && j < g.nx; }
__device__ __forceinline__ bool is_vy(const Geom& g, int i, int j) { return i >= 1 && i < g.ny && j >= 1 && j <= g.nx; }

// Node predicates inside an LDS tile.  IN marks an interior tile: the tile
// and its whole halo lie in rows 1..ny-1 and columns 1..nx-1, so every node
// is an unknown of both components, no node is wall-adjacent and no ghost
// or wall is touched; the checks then vanish at compile time.
template <bool IN>
__device__ __forceinline__ bool ux_at(const Geom& g, int i, int j) { return IN || is_vx(g, i, j); }
template <bool IN>
__device__ __forceinline__ bool uy_at(const Geom& g, int i, int j) { return IN || is_vy(g, i, j); }

template <bool IN, typename T>
__device__ __forceinline__ T dx_at(const T* sb, const T* sp, int c, int RW, int gi, const Geom& g,
                                   const LevelC<T>& k) {
    return IN ? lx_diag_inner(sb, sp, c, RW, k) : lx_diag(sb, sp, c, RW, gi, g.ny, k);
}
template <bool IN, typename T>
__device__ __forceinline__ T dy_at(const T* sb, const T* sp, int c, int RW, int gj, const Geom& g,
                                   const LevelC<T>& k) {
    return IN ? ly_diag_inner(sb, sp, c, RW, k) : ly_diag(sb, sp, c, RW, gj, g.nx, k);
}

// tile origin (gi0, gj0) and region RW x RH: is it an interior tile?
template <int RW, int RH>
__device__ __forceinline__ bool interior_tile(const Geom& g, int gi0, int gj0) {
    return gi0 >= 1 && gj0 >= 1 && gi0 + RH <= g.ny && gj0 + RW <= g.nx;
}

// ---------------------------------------------------------------------------
// LDS tiles.  A tile of TW x TH nodes (origin (i0, j0) = (1 + tby TH,
// 1 + tbx TW)) is held with a halo of H nodes: the iterate (sx, sy) and the
// viscosities (sb, sp).  The right-hand side r is only ever needed at the
// node being updated, so it is read from memory there and takes no LDS.
// ---------------------------------------------------------------------------
template <int RH>
constexpr int prolong_rows() { return RH / 2 + 4; }

// Every Gauss-Seidel / Jacobi LDS tile kernel runs kTileThreads threads.
// Loops over a tile region have a compile-time trip count and are unrolled
// with all global loads of a phase issued into registers before the first
// one is used: a tile is latency-bound (few waves per CU at the finest
// level, a handful of tiles on the small ones), and a load loop that waited
// for each load before issuing the next would serialise one memory latency
// per iteration.  512 threads: each colour stage of a small-level tile is
// then one node per thread, which shortens the dependent chain of a launch;
// the 1024^2 solve ran 5 % faster than with 256 threads (1024 threads were
// slower again), with bitwise the same results, since nodes of one stage
// are independent of each other.
constexpr int kTileThreads = 512;
// Waves per SIMD the one-sweep tile kernels ask for: 8, so that four workgroups
// share a CU and the 1024 tiles of a 1024^2 level run in one round.  The FP32 sweep
// with prolongation gets there with 61 registers (66 by itself, three workgroups per
// CU and a second, nearly empty round: 16.6 us, now 16.3 from this alone).  The
// FP64 one takes 77: its 44.5 KB of LDS allow three workgroups in any case.
constexpr int kTileWaves = 8;

template <int N>
constexpr int tile_iters() { return (N + kTileThreads - 1) / kTileThreads; }

// Entries of a field at byte offsets from a tile's first entry: the pointer is
// uniform and the offset a non-negative 32-bit value, so a load takes no
// address arithmetic of its own and the offset serves every field.
template <typename V, typename T>
__device__ __forceinline__ V tile_ld(const T* __restrict__ p, unsigned off) {
    return *(const V*)((const char*)p + off);
}
template <typename T>
__device__ __forceinline__ void tile_st(T* __restrict__ p, unsigned off, T v) {
    *(T*)((char*)p + off) = v;
}
template <typename T> struct TilePair;
template <> struct TilePair<float> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct TilePair<double> { typedef double type __attribute__((ext_vector_type(2))); };

// Load the iterate (zero / from memory / from memory + prolongated coarse
// correction) and the viscosities of the region starting at (gi0, gj0).  gj0 is
// odd and columns 1, 65, .. start a segment, so two neighbouring columns are
// one aligned vector: a thread takes pairs, which halves the loads, LDS stores
// and index arithmetic of the phase and lets the two nodes of a pair share the
// coarse values they interpolate.  These passes are bound by the instructions
// they issue (some 350 vector instructions per wave in a sweep from zero, 480
// with prolongation, over 600 before): the FP32 sweep with prolongation takes
// 15.0 us on 1024^2 (17.5) and 35 on 2048^2 (43).
template <typename T, int RW, int RH, int H, int MODE, bool IN>
__device__ __forceinline__ void tile_load(const Geom& g, const Geom& gc, int gi0, int gj0, const T* __restrict__ exi,
                                          const T* __restrict__ eyi, const T* __restrict__ eb,
                                          const T* __restrict__ ep, const T* __restrict__ ecx,
                                          const T* __restrict__ ecy, T* sx, T* sy, T* sb, T* sp, T* scx, T* scy,
                                          const LevelC<T>& k) {
    using V2 = typename TilePair<T>::type;
    constexpr int HW = RW / 2, RN = HW * RH, IT = tile_iters<RN>();
    constexpr int CR = prolong_rows<RH>(), CC = prolong_rows<RW>(), ITC = tile_iters<CR * CC>();
    constexpr bool kIter = MODE != kModeZero;
    const int tid = threadIdx.x;
    const int P = g.pitch;
    const ptrdiff_t base = (ptrdiff_t)gi0 * P + gj0;
    const T *pb = eb + base, *pp = ep + base, *px = kIter ? exi + base : nullptr, *py = kIter ? eyi + base : nullptr;
    const V2 zero = {(T)0, (T)0};
    V2 vb[IT], vp[IT], vx[kIter ? IT : 1], vy[kIter ? IT : 1];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int q = tid + it * kTileThreads;
        const int a = q / HW, m = q - (q / HW) * HW;
        const int gi = gi0 + a, gj = gj0 + 2 * m;
        // columns 0 .. nx + 1 hold entries; the pairs (-1, 0) and (nx + 1, nx + 2) hold one each (their
        // other half is padding, zero here)
        const bool in = q < RN && (IN || (gi >= 0 && gi <= g.ny + 1 && gj >= -1 && gj <= g.nx + 1));
        // (lanes without a pair repeat the tile's first own one)
        const unsigned off = (unsigned)(in ? a * P + 2 * m : H * P + H) * (unsigned)sizeof(T);
        vb[it] = tile_ld<V2>(pb, off);
        vp[it] = tile_ld<V2>(pp, off);
        if (kIter) {
            vx[it] = tile_ld<V2>(px, off);
            vy[it] = tile_ld<V2>(py, off);
        }
    }
    // first coarse row / column of the prolongation window: floor(gi0 / 2) - 1
    // (gi0 may be negative; the +64 keeps the shift on a non-negative value)
    const int ci0 = ((gi0 + 64) >> 1) - 32 - 1;
    const int cj0 = ((gj0 + 64) >> 1) - 32 - 1;
    if (MODE == kModeProlong) {
        const int Pc = gc.pitch;
        const T *qx = ecx + ((ptrdiff_t)ci0 * Pc + cj0), *qy = ecy + ((ptrdiff_t)ci0 * Pc + cj0);
        T wx[ITC], wy[ITC];
#pragma unroll
        for (int it = 0; it < ITC; ++it) {
            const int q = tid + it * kTileThreads;
            const int a = q / CC, b = q - (q / CC) * CC;
            const int I = ci0 + a, J = cj0 + b;
            const bool in = q < CR * CC && I >= 0 && I <= gc.ny + 1 && J >= 0 && J <= gc.nx + 1;
            wx[it] = wy[it] = (T)0;
            if (in) {
                const unsigned off = (unsigned)(a * Pc + b) * (unsigned)sizeof(T);
                wx[it] = tile_ld<T>(qx, off);
                wy[it] = tile_ld<T>(qy, off);
            }
        }
#pragma unroll
        for (int it = 0; it < ITC; ++it) {
            const int q = tid + it * kTileThreads;
            if (q < CR * CC) {
                scx[q] = wx[it];
                scy[q] = wy[it];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int q = tid + it * kTileThreads;
        if (q >= RN) continue;
        const int a = q / HW, m = q - (q / HW) * HW;
        if (!IN) {
            const int gi = gi0 + a, gj = gj0 + 2 * m;
            const bool row = gi >= 0 && gi <= g.ny + 1;
            const bool lo = row && gj >= 0 && gj <= g.nx + 1, hi = row && gj >= -1 && gj <= g.nx;
            vb[it] = V2{lo ? vb[it].x : (T)0, hi ? vb[it].y : (T)0};
            vp[it] = V2{lo ? vp[it].x : (T)0, hi ? vp[it].y : (T)0};
            if (kIter) {
                vx[it] = V2{lo ? vx[it].x : (T)0, hi ? vx[it].y : (T)0};
                vy[it] = V2{lo ? vy[it].x : (T)0, hi ? vy[it].y : (T)0};
            }
        }
        ((V2*)sb)[q] = vb[it];
        ((V2*)sp)[q] = vp[it];
        if (MODE == kModeZero) {
            ((V2*)sx)[q] = zero;
            ((V2*)sy)[q] = zero;
        } else {
            V2 ux = vx[it], uy = vy[it];
            if (MODE == kModeProlong) {
                // bilinear, the weights of k_prolong_add (coarse ghosts hold mirrored values); coarse
                // rows and columns relative to the LDS window.  Columns gj = 2M + 1 (between
                // coarse lines M, M + 1 for vx) and gj + 1 (on line M + 1).
                const int gi = gi0 + a, gj = gj0 + 2 * m;
                const int M = ((gj + 63) >> 1) - 32;                                // (gj - 1) / 2
                const int odd = gi & 1, I0 = (gi + 1) >> 1, I1 = odd ? I0 - 1 : I0 + 1, I = gi >> 1;
                const T* x0 = scx + ((I0 - ci0) * CC + (M - cj0));
                const T* x1 = scx + ((I1 - ci0) * CC + (M - cj0));
                const T n0 = x0[0], n1 = x0[1], f0 = x1[0], f1 = x1[1];
                const T* y0 = scy + ((I - ci0) * CC + (M - cj0));
                const T* y1 = y0 + (odd ? CC : 0);
                const T w = y0[0] + y1[0], c = y0[1] + y1[1], e = y0[2] + y1[2];    // columns M, M + 1, M + 2
                const T px0 = fma_((T)0.375, n0 + n1, (T)0.125 * (f0 + f1));
                const T px1 = fma_((T)0.75, n1, (T)0.25 * f1);
                const T py0 = fma_((T)0.375, c, (T)0.125 * w), py1 = fma_((T)0.375, c, (T)0.125 * e);
                if (ux_at<IN>(g, gi, gj)) ux.x += px0;
                if (ux_at<IN>(g, gi, gj + 1)) ux.y += px1;
                if (uy_at<IN>(g, gi, gj)) uy.x += py0;
                if (uy_at<IN>(g, gi, gj + 1)) uy.y += py1;
            }
            ((V2*)sx)[q] = ux;
            ((V2*)sy)[q] = uy;
        }
    }
    __syncthreads();
    if (MODE == kModeProlong && !IN) {
        // ghosts mirror the corrected interior values
        constexpr int RN1 = RW * RH, IT1 = tile_iters<RN1>();
#pragma unroll
        for (int it = 0; it < IT1; ++it) {
            const int q = tid + it * kTileThreads;
            if (q >= RN1) continue;
            const int a = q / RW, b = q - (q / RW) * RW;
            const int gi = gi0 + a, gj = gj0 + b;
            if (gj >= 1 && gj < g.nx) {
                if (gi == 0 && a + 1 < RH) sx[q] = k.mirS * sx[q + RW];
                if (gi == g.ny + 1 && a >= 1) sx[q] = k.mirN * sx[q - RW];
            }
            if (gi >= 1 && gi < g.ny) {
                if (gj == 0 && b + 1 < RW) sy[q] = k.mirW * sy[q + 1];
                if (gj == g.nx + 1 && b >= 1) sy[q] = k.mirE * sy[q - 1];
            }
        }
        __syncthreads();
    }
}

// Shape of the colour stages of a tile: stage s (component (s >> 1) & 1,
// colour s & 1, i.e. vx red, vx black, vy red, vy black, repeated) updates
// the nodes within h = H - 1 - s of the tile; thread t takes the nodes
// t, t + kTileThreads, ... of the stage's list (rows x half, one colour per row).
template <int TW, int TH, int H, int NSTAGE>
struct Stages {
    static constexpr int rows(int s) { return TH + 2 * (H - 1 - s); }
    static constexpr int half(int s) { return (TW + 2 * (H - 1 - s)) / 2; }
    static constexpr int iters(int s) { return (rows(s) * half(s) + kTileThreads - 1) / kTileThreads; }
    static constexpr int offset(int s) {
        int o = 0;
        for (int q = 0; q < s; ++q) o += iters(q);
        return o;
    }
    static constexpr int total() { return offset(NSTAGE); }
};

// LDS coordinates (a, b) of item q of stage s
template <int TW, int TH, int H>
__device__ __forceinline__ void stage_node(int s, int q, int gi0, int gj0, int& a, int& b) {
    const int h = H - 1 - s, col = s & 1;
    const int half = (TW + 2 * h) / 2;
    const int ar = q / half, bb = q - (q / half) * half;
    const int a0 = H - h, b0 = H - h;
    a = a0 + ar;
    const int p0 = (gi0 + a + gj0 + b0) & 1;
    b = b0 + 2 * bb + (col ^ p0);
}

// right-hand side of every node this thread updates, in stage order
template <typename T, int TW, int TH, int H, int NSTAGE, bool IN>
__device__ __forceinline__ void stage_rhs(const Geom& g, int gi0, int gj0, const T* __restrict__ rx,
                                          const T* __restrict__ ry, T* rr) {
    using S = Stages<TW, TH, H, NSTAGE>;
    const int tid = threadIdx.x;
    const int P = g.pitch;
    const T *px = rx + ((ptrdiff_t)gi0 * P + gj0), *py = ry + ((ptrdiff_t)gi0 * P + gj0);
#pragma unroll
    for (int s = 0; s < NSTAGE; ++s) {
        const int comp = (s >> 1) & 1;
#pragma unroll
        for (int it = 0; it < S::iters(s); ++it) {
            const int q = tid + it * kTileThreads;
            int a, b;
            stage_node<TW, TH, H>(s, q, gi0, gj0, a, b);
            const int gi = gi0 + a, gj = gj0 + b;
            const bool ok = q < S::rows(s) * S::half(s) && (comp == 0 ? ux_at<IN>(g, gi, gj) : uy_at<IN>(g, gi, gj));
            rr[S::offset(s) + it] = (T)0;
            if (ok) rr[S::offset(s) + it] = tile_ld<T>(comp == 0 ? px : py, (unsigned)(a * P + b) * (unsigned)sizeof(T));
        }
    }
}

// NSTAGE colour half-sweeps.  Each stage needs the previous one's values
// one node further out, hence the shrinking regions.  With GHOSTS a
// wall-adjacent node refreshes its own ghost right away; only that node
// reads the ghost, so a later sweep (or the residual) in the same pass sees
// the mirror of the latest value, as a sweep over the whole grid with
// ghosts refilled between sweeps does.  A single sweep without residual
// never re-reads a ghost, and the store writes the ghosts.  With ZERO the
// pass starts from a zero iterate, so in the first sweep the vx-red stage
// reads only zeros (L e = 0) and the vx-black and vy-red stages read no
// non-zero vy: their stencils skip those terms (fewer loads; the same values
// up to rounding).
template <typename T, int TW, int TH, int H, int NSTAGE, bool IN, bool GHOSTS, bool ZERO>
__device__ __forceinline__ void gs_stages(const Geom& g, int gi0, int gj0, T* sx, T* sy, const T* sb, const T* sp,
                                          const T* rr, T omega, const LevelC<T>& k) {
    using S = Stages<TW, TH, H, NSTAGE>;
    constexpr int RW = TW + 2 * H, RH = TH + 2 * H;
    int tid = threadIdx.x;
    // Two sweeps: the indices anew, instead of those of all eight stages kept since the loads (129 registers with 64 x 16
    // FP32 nodes from zero, one workgroup a CU; 88 without, and 32 instead of 66 with 32 x 8: 2 + 2 sweeps at
    // 1024^2 10.9 -> 8.7 ms for 48 V-cycles).
    if (NSTAGE > 4) asm("" : "+v"(tid));
#pragma unroll
    for (int s = 0; s < NSTAGE; ++s) {
        const int comp = (s >> 1) & 1;
#pragma unroll
        for (int it = 0; it < S::iters(s); ++it) {
            const int q = tid + it * kTileThreads;
            if (q >= S::rows(s) * S::half(s)) continue;
            int a, b;
            stage_node<TW, TH, H>(s, q, gi0, gj0, a, b);
            const int gi = gi0 + a, gj = gj0 + b;
            const int c = a * RW + b;
            const T r = rr[S::offset(s) + it];
            if (comp == 0) {
                if (!ux_at<IN>(g, gi, gj)) continue;
                const T d = dx_at<IN>(sb, sp, c, RW, gi, g, k);
                T e;
                if (ZERO && s == 0) e = relax((T)0, omega, r, d);
                else if (ZERO && s == 1) e = relax(sx[c], omega, r - lx_row_novy(sx, sb, sp, c, RW, k.idx, k.idy), d);
                else e = relax(sx[c], omega, r - lx_row(sx, sy, sb, sp, c, RW, k.idx, k.idy), d);
                sx[c] = e;
                if (GHOSTS && !IN) {
                    if (gi == 1 && a >= 1) sx[c - RW] = k.mirS * e;
                    if (gi == g.ny && a + 1 < RH) sx[c + RW] = k.mirN * e;
                }
            } else {
                if (!uy_at<IN>(g, gi, gj)) continue;
                const T d = dy_at<IN>(sb, sp, c, RW, gj, g, k);
                const T e = (ZERO && s == 2) ? relax((T)0, omega, r - ly_row_novy(sx, sb, c, RW, k.idx, k.idy), d)
                                             : relax(sy[c], omega, r - ly_row(sx, sy, sb, sp, c, RW, k.idx, k.idy), d);
                sy[c] = e;
                if (GHOSTS && !IN) {
                    if (gj == 1 && b >= 1) sy[c - 1] = k.mirW * e;
                    if (gj == g.nx && b + 1 < RW) sy[c + 1] = k.mirE * e;
                }
            }
        }
        __syncthreads();
    }
}

// write the tile's own nodes (and the ghosts they own) to memory
template <typename T, int TW, int TH, int H, bool IN>
__device__ __forceinline__ void tile_store(const Geom& g, int gi0, int gj0, const T* sx, const T* sy,
                                           T* __restrict__ exo, T* __restrict__ eyo, const LevelC<T>& k) {
    constexpr int RW = TW + 2 * H;
    constexpr unsigned Z = sizeof(T);
    const int P = g.pitch;
    T *px = exo + ((ptrdiff_t)gi0 * P + gj0), *py = eyo + ((ptrdiff_t)gi0 * P + gj0);
#pragma unroll
    for (int it = 0; it < tile_iters<TW * TH>(); ++it) {
        const int q = threadIdx.x + it * kTileThreads;
        if (q >= TW * TH) continue;
        const int a = H + q / TW, b = H + (q - (q / TW) * TW);
        const int gi = gi0 + a, gj = gj0 + b;
        const int c = a * RW + b;
        const unsigned off = (unsigned)(a * P + b) * Z;
        if (ux_at<IN>(g, gi, gj)) {
            const T e = sx[c];
            tile_st(px, off, e);
            if (!IN && gi == 1) tile_st(px, off - P * Z, k.mirS * e);
            if (!IN && gi == g.ny) tile_st(px, off + P * Z, k.mirN * e);
        }
        if (uy_at<IN>(g, gi, gj)) {
            const T e = sy[c];
            tile_st(py, off, e);
            if (!IN && gj == 1) tile_st(py, off - Z, k.mirW * e);
            if (!IN && gj == g.nx) tile_st(py, off + Z, k.mirE * e);
        }
    }
}

// normalised restriction of the fine residual held in LDS (stx, sty of
// row length RC, first row / column fi0, fj0) to coarse cell (I, J)
// (gather form of Alg. "4-Color Parallel Restriction", factor 2)
template <typename T, int RC>
__device__ __forceinline__ void restrict_cell(const Geom& g, const Geom& gc, const T* stx, const T* sty, int fi0,
                                              int fj0, int I, int J, T* __restrict__ rcx, T* __restrict__ rcy) {
    const int C = I * gc.pitch + J;
    if (J < gc.nx) {
        T s = (T)0, wy = (T)0;
        for (int a4 = 0; a4 < 4; ++a4) {
            const int i = 2 * I - 2 + a4;
            if (i < 1 || i > g.ny) continue;
            const T w = (a4 == 1 || a4 == 2) ? (T)0.75 : (T)0.25;
            const int c = (i - fi0) * RC + (2 * J - fj0);
            s += w * ((T)0.5 * stx[c - 1] + stx[c] + (T)0.5 * stx[c + 1]);
            wy += w;
        }
        rcx[C] = s / ((T)2 * wy);
    }
    if (I < gc.ny) {
        T s = (T)0, wx = (T)0;
        for (int b4 = 0; b4 < 4; ++b4) {
            const int j = 2 * J - 2 + b4;
            if (j < 1 || j > g.nx) continue;
            const T w = (b4 == 1 || b4 == 2) ? (T)0.75 : (T)0.25;
            const int c = (2 * I - fi0) * RC + (j - fj0);
            s += w * ((T)0.5 * sty[c - RC] + sty[c] + (T)0.5 * sty[c + RC]);
            wx += w;
        }
        rcy[C] = s / ((T)2 * wx);
    }
}

// Gauss-Seidel on an LDS tile: NS full sweeps in one pass (halo 4 NS), the
// first from zero, from the iterate in memory, or from the iterate plus the
// prolongated coarse correction (MODE).  The tile reads the old iterate and
// writes its own nodes to the other buffer, so overlapping tiles never see
// each other's new values and the result equals NS sweeps over the whole
// grid exactly.  With RR the pass continues (halo 4 NS + 2) with the
// residual r - L e on the tile grown by one node and the restriction of the
// coarse cells the tile covers (TW x TH fine = TW/2 x TH/2 coarse): the
// down leg of a V-cycle level in one launch, the fine residual never going
// to memory.
template <typename T, int TW, int TH, int NS, int MODE, int RR, bool IN>
__device__ __forceinline__ void gs_tile_run(const Geom& g, const Geom& gc, const T* __restrict__ exi,
                                            const T* __restrict__ eyi, T* __restrict__ exo, T* __restrict__ eyo,
                                            const T* __restrict__ rx, const T* __restrict__ ry,
                                            const T* __restrict__ eb, const T* __restrict__ ep,
                                            const T* __restrict__ ecx, const T* __restrict__ ecy,
                                            T* __restrict__ rcx, T* __restrict__ rcy, T omega, int tbx, int tby,
                                            T* sx, T* sy, T* sb, T* sp, T* scx, T* scy, T* stx, T* sty) {
    constexpr int H = 4 * NS + (RR ? 2 : 0);
    constexpr int RW = TW + 2 * H, RH = TH + 2 * H;
    constexpr int TRW = RR ? TW + 2 : 1, TRH = RR ? TH + 2 : 1;
    constexpr int NR = Stages<TW, TH, H, 4 * NS>::total();
    constexpr int ITR = RR ? tile_iters<TRW * TRH>() : 1;
    const int i0 = 1 + tby * TH, j0 = 1 + tbx * TW;
    const int gi0 = i0 - H, gj0 = j0 - H;
    const int P = g.pitch;
    const LevelC<T> k = level_consts<T>(g);
    // right-hand sides first: they are in flight while the tile loads
    T rr[NR];
    stage_rhs<T, TW, TH, H, 4 * NS, IN>(g, gi0, gj0, rx, ry, rr);
    T rrx[ITR], rry[ITR];
    if (RR) {
#pragma unroll
        for (int it = 0; it < ITR; ++it) {
            const int q = threadIdx.x + it * kTileThreads;
            const int a = q / TRW, b = q - (q / TRW) * TRW;
            const int gi = i0 - 1 + a, gj = j0 - 1 + b;
            const bool okx = q < TRW * TRH && ux_at<IN>(g, gi, gj), oky = q < TRW * TRH && uy_at<IN>(g, gi, gj);
            const unsigned off = (unsigned)(a * P + b) * (unsigned)sizeof(T);
            const ptrdiff_t base = (ptrdiff_t)(i0 - 1) * P + (j0 - 1);
            rrx[it] = rry[it] = (T)0;
            if (okx) rrx[it] = tile_ld<T>(rx + base, off);
            if (oky) rry[it] = tile_ld<T>(ry + base, off);
        }
    }
    tile_load<T, RW, RH, H, MODE, IN>(g, gc, gi0, gj0, exi, eyi, eb, ep, ecx, ecy, sx, sy, sb, sp, scx, scy, k);
    gs_stages<T, TW, TH, H, 4 * NS, IN, (NS > 1 || RR), MODE == kModeZero>(g, gi0, gj0, sx, sy, sb, sp, rr, omega,
                                                                          k);
    tile_store<T, TW, TH, H, IN>(g, gi0, gj0, sx, sy, exo, eyo, k);
    if (RR) {
#pragma unroll
        for (int it = 0; it < ITR; ++it) {
            const int q = threadIdx.x + it * kTileThreads;
            if (q >= TRW * TRH) continue;
            const int a = q / TRW, b = q - (q / TRW) * TRW;
            const int gi = i0 - 1 + a, gj = j0 - 1 + b;
            const int c = (a + H - 1) * RW + (b + H - 1);
            stx[q] = ux_at<IN>(g, gi, gj) ? rrx[it] - lx_row(sx, sy, sb, sp, c, RW, k.idx, k.idy) : (T)0;
            sty[q] = uy_at<IN>(g, gi, gj) ? rry[it] - ly_row(sx, sy, sb, sp, c, RW, k.idx, k.idy) : (T)0;
        }
        __syncthreads();
        const int I0 = 1 + tby * (TH / 2), J0 = 1 + tbx * (TW / 2);
#pragma unroll
        for (int it = 0; it < tile_iters<(TH / 2) * (TW / 2)>(); ++it) {
            const int q = threadIdx.x + it * kTileThreads;
            if (q >= (TH / 2) * (TW / 2)) continue;
            const int I = I0 + q / (TW / 2), J = J0 + (q - (q / (TW / 2)) * (TW / 2));
            if (I > gc.ny || J > gc.nx) continue;
            restrict_cell<T, TRW>(g, gc, stx, sty, i0 - 1, j0 - 1, I, J, rcx, rcy);
        }
    }
}

template <typename T, int TW, int TH, int NS, int MODE, int RR>
__device__ __forceinline__ void gs_tile_body(const Geom& g, const Geom& gc, const T* __restrict__ exi,
                                             const T* __restrict__ eyi, T* __restrict__ exo, T* __restrict__ eyo,
                                             const T* __restrict__ rx, const T* __restrict__ ry,
                                             const T* __restrict__ eb, const T* __restrict__ ep,
                                             const T* __restrict__ ecx, const T* __restrict__ ecy,
                                             T* __restrict__ rcx, T* __restrict__ rcy, T omega, int tbx, int tby) {
    static_assert(TW % 2 == 0 && TH % 2 == 0, "tiles cover whole coarse cells");
    static_assert(!(RR && MODE == kModeProlong), "the down leg starts from zero or an iterate");
    constexpr int H = 4 * NS + (RR ? 2 : 0);
    constexpr int RW = TW + 2 * H, RH = TH + 2 * H, RN = RW * RH;
    constexpr int CN = MODE == kModeProlong ? prolong_rows<RH>() * prolong_rows<RW>() : 1;
    constexpr int TRW = RR ? TW + 2 : 1, TRH = RR ? TH + 2 : 1;
    static_assert((4 * RN + 2 * CN + 2 * TRW * TRH) * sizeof(T) <= 65536, "tile exceeds 64 KB of LDS");
    __shared__ __align__(16) T sx[RN], sy[RN], sb[RN], sp[RN];
    __shared__ T scx[CN], scy[CN];
    __shared__ T stx[TRW * TRH], sty[TRW * TRH];
    // uniform per tile: interior tiles take the check-free path
    if (interior_tile<RW, RH>(g, 1 + tby * TH - H, 1 + tbx * TW - H))
        gs_tile_run<T, TW, TH, NS, MODE, RR, true>(g, gc, exi, eyi, exo, eyo, rx, ry, eb, ep, ecx, ecy, rcx, rcy,
                                                   omega, tbx, tby, sx, sy, sb, sp, scx, scy, stx, sty);
    else
        gs_tile_run<T, TW, TH, NS, MODE, RR, false>(g, gc, exi, eyi, exo, eyo, rx, ry, eb, ep, ecx, ecy, rcx, rcy,
                                                    omega, tbx, tby, sx, sy, sb, sp, scx, scy, stx, sty);
}

// one damped Jacobi sweep on an LDS tile (halo 2: one node would do, an even
// halo keeps the region's columns in aligned pairs)
template <typename T, int TW, int TH, int MODE>
__device__ __forceinline__ void jacobi_tile_body(const Geom& g, const Geom& gc, const T* __restrict__ exi,
                                                 const T* __restrict__ eyi, T* __restrict__ exo,
                                                 T* __restrict__ eyo, const T* __restrict__ rx,
                                                 const T* __restrict__ ry, const T* __restrict__ eb,
                                                 const T* __restrict__ ep, const T* __restrict__ ecx,
                                                 const T* __restrict__ ecy, T omega, int tbx, int tby) {
    constexpr int H = 2;
    constexpr int RW = TW + 2 * H, RH = TH + 2 * H, RN = RW * RH;
    constexpr int CN = MODE == kModeProlong ? prolong_rows<RH>() * prolong_rows<RW>() : 1;
    __shared__ __align__(16) T sx[RN], sy[RN], sb[RN], sp[RN];
    __shared__ T scx[CN], scy[CN];
    constexpr int IT = tile_iters<TW * TH>();
    const int i0 = 1 + tby * TH, j0 = 1 + tbx * TW;
    const int gi0 = i0 - H, gj0 = j0 - H;
    const int P = g.pitch;
    const LevelC<T> k = level_consts<T>(g);
    T rrx[IT], rry[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int q = threadIdx.x + it * kTileThreads;
        const int a = H + q / TW, b = H + (q - (q / TW) * TW);
        const int gi = gi0 + a, gj = gj0 + b;
        rrx[it] = q < TW * TH && is_vx(g, gi, gj) ? rx[gi * P + gj] : (T)0;
        rry[it] = q < TW * TH && is_vy(g, gi, gj) ? ry[gi * P + gj] : (T)0;
    }
    tile_load<T, RW, RH, H, MODE, false>(g, gc, gi0, gj0, exi, eyi, eb, ep, ecx, ecy, sx, sy, sb, sp, scx, scy, k);
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int q = threadIdx.x + it * kTileThreads;
        if (q >= TW * TH) continue;
        const int a = H + q / TW, b = H + (q - (q / TW) * TW);
        const int gi = gi0 + a, gj = gj0 + b;
        const int c = a * RW + b;
        const int cg = gi * P + gj;
        if (is_vx(g, gi, gj)) {
            const T d = lx_diag(sb, sp, c, RW, gi, g.ny, k);
            const T e = relax(sx[c], omega, rrx[it] - lx_row(sx, sy, sb, sp, c, RW, k.idx, k.idy), d);
            exo[cg] = e;
            if (gi == 1) exo[cg - P] = k.mirS * e;
            if (gi == g.ny) exo[cg + P] = k.mirN * e;
        }
        if (is_vy(g, gi, gj)) {
            const T d = ly_diag(sb, sp, c, RW, gj, g.nx, k);
            const T e = relax(sy[c], omega, rry[it] - ly_row(sx, sy, sb, sp, c, RW, k.idx, k.idy), d);
            eyo[cg] = e;
            if (gj == 1) eyo[cg - 1] = k.mirW * e;
            if (gj == g.nx) eyo[cg + 1] = k.mirE * e;
        }
    }
}

// one smoothing sweep on an LDS tile (either smoother)
template <typename T, int TW, int TH, int SM, int MODE>
__device__ __forceinline__ void smooth_tile_body(const Geom& g, const Geom& gc, const T* __restrict__ exi,
                                                 const T* __restrict__ eyi, T* __restrict__ exo,
                                                 T* __restrict__ eyo, const T* __restrict__ rx,
                                                 const T* __restrict__ ry, const T* __restrict__ eb,
                                                 const T* __restrict__ ep, const T* __restrict__ ecx,
                                                 const T* __restrict__ ecy, T omega, int tbx, int tby) {
    if (SM == kSmGS)
        gs_tile_body<T, TW, TH, 1, MODE, 0>(g, gc, exi, eyi, exo, eyo, rx, ry, eb, ep, ecx, ecy, nullptr, nullptr,
                                            omega, tbx, tby);
    else
        jacobi_tile_body<T, TW, TH, MODE>(g, gc, exi, eyi, exo, eyo, rx, ry, eb, ep, ecx, ecy, omega, tbx, tby);
}

// ---------------------------------------------------------------------------
// fused residual + restriction
// ---------------------------------------------------------------------------
template <typename T, int CTW, int CTH>
__device__ __forceinline__ void res_restrict_body(const Geom& g, const Geom& gc, const T* __restrict__ ex,
                                                  const T* __restrict__ ey, const T* __restrict__ rx,
                                                  const T* __restrict__ ry, const T* __restrict__ eb,
                                                  const T* __restrict__ ep, T* __restrict__ rcx,
                                                  T* __restrict__ rcy, int tbx, int tby) {
    constexpr int NT = CTW * CTH;
    constexpr int RR = 2 * CTH + 2, RC = 2 * CTW + 2;   // fine residual footprint
    constexpr int LR = RR + 2, LC = RC + 2;             // loaded region
    constexpr int LN = LR * LC, RN = RR * RC;
    __shared__ T sx[LN], sy[LN], sb[LN], sp[LN], stx[RN], sty[RN];
    const int tid = threadIdx.x;
    const int I0 = 1 + tby * CTH, J0 = 1 + tbx * CTW;
    const int fi0 = 2 * I0 - 2, fj0 = 2 * J0 - 2;       // first residual row / column
    const int li0 = fi0 - 1, lj0 = fj0 - 1;             // first loaded row / column
    const int P = g.pitch;
    const LevelC<T> k = level_consts<T>(g);
    constexpr int ITL = (LN + NT - 1) / NT, ITR = (RN + NT - 1) / NT;
    // every load of the tile in flight before the first use (see kTileThreads)
    T vx[ITL], vy[ITL], vb[ITL], vp[ITL], rrx[ITR], rry[ITR];
    const ptrdiff_t rbase = (ptrdiff_t)fi0 * P + fj0, lbase = (ptrdiff_t)li0 * P + lj0;
    const T *prx = rx + rbase, *pry = ry + rbase, *px = ex + lbase, *py = ey + lbase, *pb = eb + lbase, *pp = ep + lbase;
#pragma unroll
    for (int it = 0; it < ITR; ++it) {
        const int q = tid + it * NT;
        const int a = q / RC, b = q - (q / RC) * RC;
        const int gi = fi0 + a, gj = fj0 + b;
        const unsigned off = (unsigned)(a * P + b) * (unsigned)sizeof(T);
        rrx[it] = rry[it] = (T)0;
        if (q < RN && is_vx(g, gi, gj)) rrx[it] = tile_ld<T>(prx, off);
        if (q < RN && is_vy(g, gi, gj)) rry[it] = tile_ld<T>(pry, off);
    }
#pragma unroll
    for (int it = 0; it < ITL; ++it) {
        const int q = tid + it * NT;
        const int a = q / LC, b = q - (q / LC) * LC;
        const int gi = li0 + a, gj = lj0 + b;
        const bool in = q < LN && gi >= 0 && gi <= g.ny + 1 && gj >= 0 && gj <= g.nx + 1;
        const unsigned off = (unsigned)(a * P + b) * (unsigned)sizeof(T);
        vx[it] = vy[it] = vb[it] = vp[it] = (T)0;
        if (in) {
            vx[it] = tile_ld<T>(px, off);
            vy[it] = tile_ld<T>(py, off);
            vb[it] = tile_ld<T>(pb, off);
            vp[it] = tile_ld<T>(pp, off);
        }
    }
#pragma unroll
    for (int it = 0; it < ITL; ++it) {
        const int q = tid + it * NT;
        if (q >= LN) continue;
        sx[q] = vx[it];
        sy[q] = vy[it];
        sb[q] = vb[it];
        sp[q] = vp[it];
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITR; ++it) {
        const int q = tid + it * NT;
        if (q >= RN) continue;
        const int a = q / RC, b = q - (q / RC) * RC;
        const int gi = fi0 + a, gj = fj0 + b;
        const int cl = (a + 1) * LC + (b + 1);
        stx[q] = is_vx(g, gi, gj) ? rrx[it] - lx_row(sx, sy, sb, sp, cl, LC, k.idx, k.idy) : (T)0;
        sty[q] = is_vy(g, gi, gj) ? rry[it] - ly_row(sx, sy, sb, sp, cl, LC, k.idx, k.idy) : (T)0;
    }
    __syncthreads();
    const int I = I0 + tid / CTW, J = J0 + (tid - (tid / CTW) * CTW);
    if (I > gc.ny || J > gc.nx) return;
    restrict_cell<T, RC>(g, gc, stx, sty, fi0, fj0, I, J, rcx, rcy);
}

template <typename T>
constexpr int tile_h() { return sizeof(T) == 4 ? 16 : 8; }
// coarse cells per fused residual + restriction tile: kRRTileW x rr_tile_h
// (one thread each; 32 x 8 for either type: taller FP32 tiles gained nothing,
// 32 x 4 FP64 tiles were 2 % slower per solve)
template <typename T>
constexpr int rr_tile_h() { return 8; }
constexpr int kTileW = 64;
constexpr int kRRTileW = 32;

}  // namespace dev
}  // namespace tph
