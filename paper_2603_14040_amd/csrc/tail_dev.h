// Coarse tail of the V-cycle in one workgroup: every level from a small one
// (at most 64 x 64 cells) down to the coarsest, ending in the FP64 dense
// solve.  Shared by the single-problem kernel (fused.hip) and the batched one
// (batch.hip).
//
// What bounds it: one workgroup on one compute unit, a chain of dependent
// phases (four colours per Gauss-Seidel sweep, residual, restriction, dense
// solve, prolongation) with a barrier after each.  Memory does not matter;
// the instructions issued per phase by the waves that share a SIMD do, and
// the LDS latency at the head of each phase.  Hence:
//   * A thread owns the two horizontally adjacent cells (i, 2m+1), (i, 2m+2)
//     of a level (every smoothed level has an even number of columns: it was
//     halved), one of them red and one black, so each colour phase updates
//     exactly one node per owned pair and no lane idles for its colour.
//   * A pair's viscosities, right-hand side and diagonals (in FP32 their
//     reciprocals) are put into registers once per visit of a level; a phase
//     reads only the iterate.
//   * Both components of a node share one LDS word pair, and rows are stored
//     split by column parity, so the stride-2 accesses of a colour phase touch
//     consecutive words.  Addresses are byte addresses, kept per cell.
//   * Waves without a pair on a (coarser) level go straight to the barrier.
//   * On the top level the residual overwrites the iterate in LDS while the
//     owned values wait in registers, and its viscosities and right-hand side
//     never enter LDS.
// Every node goes through the operations of the level-by-level kernels in their
// order (lx_row, relax, restrict_cell, the bilinear prolongation and their mirrors, the
// dense product by 16 lanes a row), so the cycle gives the same bits.
// Measured, one launch, 32 x 32 top, three levels: FP32 17 us with 1 + 1 sweeps
// (27 us with a thread per node, its stencil read from LDS in every phase), 18 us
// with 2 + 2 (36); FP64 24 us with 2 + 2 (47).
// Registers: 222 to 282, one or two waves a SIMD; the shapes of two and four pairs a thread in
// FP64 and FP32 spill 18 and 8 of them (22 and 2 in the batch).
// KP pairs per thread cover the top level; the levels below it have a quarter
// of its cells, so one pair per thread covers them.
#pragma once
#include "kernels.h"
#include "reduce.h"
#include "stencil.h"

namespace tph {
namespace dev {

template <typename T> struct TailVec;
template <> struct TailVec<float> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct TailVec<double> { typedef double type __attribute__((ext_vector_type(2))); };
// both components of a node (x: vx, y: vy), or two neighbouring columns of a field
template <typename T> using TailV2 = typename TailVec<T>::type;

// a * b + c * d as the compiler contracts it in the level-by-level kernels: the
// first product inside the fused multiply-add.  Spelled out, because which one
// it picks depends on the order of the loads around it.
__device__ __forceinline__ float tail_fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double tail_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }

// LDS by byte address: the compiler then adds nothing to an address it is given
#define TPH_LDS __attribute__((address_space(3)))
template <typename V>
__device__ __forceinline__ V lds_ld(unsigned a) { return *(const TPH_LDS V*)a; }
template <typename V>
__device__ __forceinline__ void lds_st(unsigned a, V v) { *(TPH_LDS V*)a = v; }

// Hides from the compiler that an address is the same in every sweep: it would
// otherwise keep every neighbour's address of every phase in a register.
__device__ __forceinline__ unsigned tail_opaque(unsigned v) {
    asm volatile("" : "+v"(v));
    return v;
}

// quotient of small non-negative integers (n < 2^20) by a reciprocal: exact, as
// (n + 1/2) / d is at least 1 / (2 d) away from an integer
__device__ __forceinline__ int small_div(int n, float rd) { return (int)(((float)n + 0.5f) * rd); }

// byte address of the word pair of node (i, j) of a level whose array starts at base
template <typename T>
__device__ __forceinline__ unsigned tail_at(const TailLevel<T>& L, unsigned base, int i, int j) {
    return base + i * L.row + (j >> 1) * (unsigned)sizeof(TailV2<T>) + ((j & 1) ? L.odd : 0u);
}

// The part of relax() that depends on the diagonal alone, and the rest of it:
// FP32 multiplies by the hardware reciprocal, FP64 divides.
__device__ __forceinline__ float tail_inv(float d) { return __builtin_amdgcn_rcpf(d); }
__device__ __forceinline__ double tail_inv(double d) { return d; }
__device__ __forceinline__ float tail_relax(float e, float omega, float res, float inv) {
    return tail_fma(omega * res, inv, e);
}
__device__ __forceinline__ double tail_relax(double e, double omega, double res, double inv) {
    return e + omega * res / inv;
}

// One owned cell in registers: the viscosities of its stencil (eta_p here, east
// and north; eta_b here, west and south), the right-hand side and the
// diagonals' part of relax().
template <typename T>
struct TailCell {
    T pc, pe, pn, bc, bw, bs;
    T ix, iy, rx, ry;
};

// A thread's pair of cells ordered red, black ((i + j) even, odd).  a: byte
// address of each; e, w: byte offsets of the red cell's east and west
// neighbours (the black cell's are -w and -e, its column having the other
// parity).  Threads beyond the last pair (live = false) repeat the first
// pair's arithmetic on a spare word pair.
template <typename T>
struct TailPair {
    int i, j0;               // row and first (odd) column
    bool live;
    unsigned a[2];
    int e, w;
    TailCell<T> q[2];
    __device__ __forceinline__ int col(int c) const { return (i & 1) == (c ^ 1) ? j0 : j0 + 1; }
    __device__ __forceinline__ int east(int c) const { return c == 0 ? e : -w; }
    __device__ __forceinline__ int west(int c) const { return c == 0 ? w : -e; }
};

// What a pair needs of its level, as loaded: eta_p of its cells and of the
// cells east and north, eta_b of its cells and of those west and south, the
// right-hand side.  Vectors hold columns j0, j0 + 1.
template <typename T>
struct TailRaw {
    TailV2<T> p, pn, b, bs, rx, ry;
    T pe, bw;
};

// pair number t of a level: its place and addresses
template <typename T>
__device__ __forceinline__ void tail_place(const TailLevel<T>& L, unsigned base, unsigned spare, int t,
                                           TailPair<T>& pr) {
    constexpr int S = sizeof(TailV2<T>);
    const int hp = L.nx >> 1;
    pr.live = t < hp * L.ny;
    const int q = pr.live ? t : 0;
    const int r = small_div(q, L.rhp);
    pr.i = 1 + r;
    pr.j0 = 1 + 2 * (q - r * hp);
    const bool odd = pr.i & 1;           // odd row: the odd column j0 is red
    const unsigned o = tail_at<T>(L, base, pr.i, pr.j0), v = tail_at<T>(L, base, pr.i, pr.j0 + 1);
    pr.a[0] = pr.live ? (odd ? o : v) : spare;
    pr.a[1] = pr.live ? (odd ? v : o) : spare;
    pr.e = odd ? S - (int)L.odd : (int)L.odd;
    pr.w = odd ? -(int)L.odd : (int)L.odd - S;
}

// The pair's cells from what was loaded.  Viscosities beyond the east and north
// walls are not defined and belong to no unknown: one there keeps the unused
// arithmetic finite.
template <typename T>
__device__ __forceinline__ void tail_finish(const TailLevel<T>& L, const TailRaw<T>& r, TailPair<T>& pr) {
    TailCell<T> q[2];
    const bool east = pr.j0 + 1 >= L.nx, north = pr.i >= L.ny;
    q[0].pc = r.p.x;
    q[1].pc = q[0].pe = r.p.y;
    q[1].pe = east ? (T)1 : r.pe;
    q[0].pn = north ? (T)1 : r.pn.x;
    q[1].pn = north ? (T)1 : r.pn.y;
    q[0].bc = q[1].bw = r.b.x;
    q[1].bc = r.b.y;
    q[0].bw = r.bw;
    q[0].bs = r.bs.x;
    q[1].bs = r.bs.y;
    q[0].rx = r.rx.x;
    q[1].rx = east ? (T)0 : r.rx.y;
    q[0].ry = north ? (T)0 : r.ry.x;
    q[1].ry = north ? (T)0 : r.ry.y;
#pragma unroll
    for (int c = 0; c < 2; ++c) {                    // lx_diag, ly_diag
        const int i = pr.i, j = pr.j0 + c;
        const T ct = (i == L.ny) ? ((T)1 - L.mirN) : (T)1, cb = (i == 1) ? ((T)1 - L.mirS) : (T)1;
        const T cr = (j == L.nx) ? ((T)1 - L.mirE) : (T)1, cl = (j == 1) ? ((T)1 - L.mirW) : (T)1;
        q[c].ix = tail_inv(tail_fma(-(T)2 * (q[c].pe + q[c].pc), L.idx2, -(tail_fma(q[c].bc, ct, q[c].bs * cb) * L.idy2)));
        q[c].iy = tail_inv(tail_fma(-(T)2 * (q[c].pn + q[c].pc), L.idy2, -(tail_fma(q[c].bc, cr, q[c].bw * cl) * L.idx2)));
    }
    const bool odd = pr.i & 1;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const TailCell<T>&u = q[c], &v = q[1 - c];
        TailCell<T>& o = pr.q[c];
        o.pc = odd ? u.pc : v.pc;
        o.pe = odd ? u.pe : v.pe;
        o.pn = odd ? u.pn : v.pn;
        o.bc = odd ? u.bc : v.bc;
        o.bw = odd ? u.bw : v.bw;
        o.bs = odd ? u.bs : v.bs;
        o.ix = odd ? u.ix : v.ix;
        o.iy = odd ? u.iy : v.iy;
        o.rx = odd ? u.rx : v.rx;
        o.ry = odd ? u.ry : v.ry;
    }
}

// (L e) of one component at an owned cell: lx_row / ly_row, the factor 2 of the
// normal stresses applied to their difference (which is exact); o: the cell's
// own values
template <typename T>
__device__ __forceinline__ T tail_lx(const TailLevel<T>& L, const TailCell<T>& q, unsigned a, int e, int w,
                                     TailV2<T> o) {
    constexpr unsigned Y = sizeof(T);
    const TailV2<T> ve = lds_ld<TailV2<T>>(a + e), vs = lds_ld<TailV2<T>>(a - L.row);
    const T xw = lds_ld<T>(a + w), xn = lds_ld<T>(a + L.row), yse = lds_ld<T>(a - L.row + e + Y);
    const T sxx = tail_fma(q.pe, (ve.x - o.x) * L.idx, -(q.pc * ((o.x - xw) * L.idx)));
    const T gt = tail_fma(xn - o.x, L.idy, (ve.y - o.y) * L.idx);
    const T gb = tail_fma(o.x - vs.x, L.idy, (yse - vs.y) * L.idx);
    return tail_fma(sxx, L.idx_2, tail_fma(q.bc, gt, -(q.bs * gb)) * L.idy);
}
template <typename T>
__device__ __forceinline__ T tail_ly(const TailLevel<T>& L, const TailCell<T>& q, unsigned a, int e, int w,
                                     TailV2<T> o) {
    constexpr unsigned Y = sizeof(T);
    const TailV2<T> vn = lds_ld<TailV2<T>>(a + L.row), vw = lds_ld<TailV2<T>>(a + w);
    const T ys = lds_ld<T>(a - L.row + Y), ye = lds_ld<T>(a + e + Y), xnw = lds_ld<T>(a + L.row + w);
    const T syy = tail_fma(q.pn, (vn.y - o.y) * L.idy, -(q.pc * ((o.y - ys) * L.idy)));
    const T gr = tail_fma(vn.x - o.x, L.idy, (ye - o.y) * L.idx);
    const T gl = tail_fma(xnw - vw.x, L.idy, (o.y - vw.y) * L.idx);
    return tail_fma(syy, L.idy_2, tail_fma(q.bc, gr, -(q.bw * gl)) * L.idx);
}
// the damped update of a component; a cell without an unknown keeps its zero
template <typename T>
__device__ __forceinline__ T tail_new_x(const TailLevel<T>& L, T om, const TailPair<T>& pr, int c, unsigned a, TailV2<T> o) {
    const TailCell<T>& q = pr.q[c];
    const T v = tail_relax(o.x, om, q.rx - tail_lx(L, q, a, pr.east(c), pr.west(c), o), q.ix);
    return pr.col(c) < L.nx ? v : o.x;
}
template <typename T>
__device__ __forceinline__ T tail_new_y(const TailLevel<T>& L, T om, const TailPair<T>& pr, int c, unsigned a, TailV2<T> o) {
    const TailCell<T>& q = pr.q[c];
    const T v = tail_relax(o.y, om, q.ry - tail_ly(L, q, a, pr.east(c), pr.west(c), o), q.iy);
    return pr.i < L.ny ? v : o.y;
}

// Store a component's value with the ghost that mirrors it; inside, the ghost
// store repeats the node's own, so that a phase has no branches.
template <typename T>
__device__ __forceinline__ void tail_put_x(const TailLevel<T>& L, const TailPair<T>& pr, unsigned a, T v) {
    const int g = !pr.live ? 0 : pr.i == 1 ? -(int)L.row : pr.i == L.ny ? (int)L.row : 0;
    const T m = pr.i == 1 ? L.mirS : pr.i == L.ny ? L.mirN : (T)1;
    lds_st<T>(a, v);
    lds_st<T>(a + g, g ? m * v : v);
}
template <typename T>
__device__ __forceinline__ void tail_put_y(const TailLevel<T>& L, const TailPair<T>& pr, int c, unsigned a, T v) {
    constexpr unsigned Y = sizeof(T);
    const int j = pr.col(c);
    const int g = !pr.live ? 0 : j == 1 ? pr.west(c) : j == L.nx ? pr.east(c) : 0;
    const T m = j == 1 ? L.mirW : j == L.nx ? L.mirE : (T)1;
    lds_st<T>(a + Y, v);
    lds_st<T>(a + g + Y, g ? m * v : v);
}

template <typename T, int K>
__device__ __forceinline__ void tail_put(const TailLevel<T>& L, const TailPair<T> (&pr)[K], const TailV2<T> (&nv)[K][2]) {
#pragma unroll
    for (int u = 0; u < K; ++u)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            tail_put_x(L, pr[u], pr[u].a[c], nv[u][c].x);
            tail_put_y(L, pr[u], c, pr[u].a[c], nv[u][c].y);
        }
}

// nu sweeps on a level, in place.  Gauss-Seidel: vx red, vx black, vy red, vy
// black, a barrier after each; Jacobi: all new values from the old iterate,
// then written.  All owned cells are read before any is written, so their loads
// are in flight together.  wave: this wave owns a pair of the level.
template <typename T, int K>
__device__ __forceinline__ void tail_smooth(const TailLevel<T>& L, T om, const TailPair<T> (&pr)[K], int nu, bool gs,
                                            bool wave) {
    for (int s = 0; s < nu; ++s) {
        if (gs) {
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const int c = h & 1;
                if (wave) {
                    T nv[K];
                    unsigned a[K];
#pragma unroll
                    for (int u = 0; u < K; ++u) {
                        a[u] = tail_opaque(pr[u].a[c]);
                        const TailV2<T> o = lds_ld<TailV2<T>>(a[u]);
                        nv[u] = h < 2 ? tail_new_x(L, om, pr[u], c, a[u], o) : tail_new_y(L, om, pr[u], c, a[u], o);
                    }
#pragma unroll
                    for (int u = 0; u < K; ++u) {
                        if (h < 2) tail_put_x(L, pr[u], a[u], nv[u]);
                        else tail_put_y(L, pr[u], c, a[u], nv[u]);
                    }
                }
                __syncthreads();
            }
        } else {
            TailV2<T> nv[K][2];
            if (wave) {
#pragma unroll
                for (int u = 0; u < K; ++u)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const unsigned a = tail_opaque(pr[u].a[c]);
                        const TailV2<T> o = lds_ld<TailV2<T>>(a);
                        nv[u][c].x = tail_new_x(L, om, pr[u], c, a, o);
                        nv[u][c].y = tail_new_y(L, om, pr[u], c, a, o);
                    }
            }
            __syncthreads();
            if (wave) tail_put(L, pr, nv);
            __syncthreads();
        }
    }
}

// the owned cells' values and their residuals r - L e (zero where a component has no unknown)
template <typename T, int K>
__device__ __forceinline__ void tail_residual(const TailLevel<T>& L, const TailPair<T> (&pr)[K], TailV2<T> (&o)[K][2],
                                              TailV2<T> (&t)[K][2]) {
#pragma unroll
    for (int u = 0; u < K; ++u)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const unsigned a = tail_opaque(pr[u].a[c]);
            o[u][c] = lds_ld<TailV2<T>>(a);
            const T rx = pr[u].q[c].rx - tail_lx(L, pr[u].q[c], a, pr[u].east(c), pr[u].west(c), o[u][c]);
            const T ry = pr[u].q[c].ry - tail_ly(L, pr[u].q[c], a, pr[u].east(c), pr[u].west(c), o[u][c]);
            t[u][c].x = pr[u].col(c) < L.nx ? rx : (T)0;
            t[u][c].y = pr[u].i < L.ny ? ry : (T)0;
        }
}

// Normalised restriction (gather form of Alg. "4-Color Parallel Restriction",
// factor 2) of the residual of level F held at base to coarse cell (I, J).
// Ghost rows and columns take weight zero and their (stale) entries are not
// read; the sum of weights is 4 inside and 3.5 at a wall.
template <typename T>
__device__ __forceinline__ T tail_weigh(T r0, T r1, T r2, T r3, bool lo, bool hi) {
    T s = lo ? (T)0.25 * r0 : (T)0;
    s = tail_fma((T)0.75, r1, s);
    s = tail_fma((T)0.75, r2, s);
    if (hi) s = tail_fma((T)0.25, r3, s);
    return lo && hi ? s * (T)0.25 : s / (lo || hi ? (T)3.5 : (T)3);
}
template <typename T>
__device__ __forceinline__ T tail_restrict_x(const TailLevel<T>& F, unsigned base, int ncy, int I, int J) {
    constexpr unsigned S = sizeof(TailV2<T>);
    // column 2J is entry J of the even half; columns 2J - 1, 2J + 1 entries J - 1, J of the odd one
    const unsigned c = base + (2 * I - 1) * F.row + J * S;
    const bool lo = I > 1, hi = I < ncy;
    auto row = [&](unsigned a) { return (T)0.5 * lds_ld<T>(a + F.odd - S) + lds_ld<T>(a) + (T)0.5 * lds_ld<T>(a + F.odd); };
    const T r0 = row(lo ? c - F.row : c), r1 = row(c), r2 = row(c + F.row), r3 = row(hi ? c + 2 * F.row : c);
    return tail_weigh(r0, r1, r2, r3, lo, hi);
}
template <typename T>
__device__ __forceinline__ T tail_restrict_y(const TailLevel<T>& F, unsigned base, int ncx, int I, int J) {
    constexpr unsigned S = sizeof(TailV2<T>), Y = sizeof(T);
    // columns 2J - 2 and 2J are entries J - 1, J of the even half; 2J - 1 and 2J + 1 entries J - 1, J of the odd one
    const unsigned c = base + 2 * I * F.row + J * S + Y;
    const bool lo = J > 1, hi = J < ncx;
    auto col = [&](unsigned a) { return (T)0.5 * lds_ld<T>(a - F.row) + lds_ld<T>(a) + (T)0.5 * lds_ld<T>(a + F.row); };
    const T c0 = col(c - S), c1 = col(c + F.odd - S), c2 = col(c), c3 = col(c + F.odd);
    return tail_weigh(c0, c1, c2, c3, lo, hi);
}

// o += P e_c on the owned cells (bilinear; zero where a component has no
// unknown), then stored; the coarse level C is held at base
template <typename T, int K>
__device__ __forceinline__ void tail_correct(const TailLevel<T>& L, const TailLevel<T>& C, unsigned base,
                                             const TailPair<T> (&pr)[K], TailV2<T> (&o)[K][2]) {
    constexpr unsigned Y = sizeof(T);
#pragma unroll
    for (int u = 0; u < K; ++u) {
        // the nearer and the farther coarse row / column of the fine one, and
        // the row / column at or below a node on a coarse line
        const int i = pr[u].i, I0 = (i + 1) >> 1, I1 = (i & 1) ? I0 - 1 : I0 + 1, I = i >> 1;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int j = pr[u].col(c), J0 = (j + 1) >> 1, J1 = (j & 1) ? J0 - 1 : J0 + 1, J = j >> 1;
            // a column on a coarse line takes that line alone (both reads hit it)
            const int Je = J + (j & 1), Ie = I + (i & 1);
            const unsigned n0 = tail_at<T>(C, base, I0, J), n1 = tail_at<T>(C, base, I0, Je);
            const unsigned f0 = tail_at<T>(C, base, I1, J), f1 = tail_at<T>(C, base, I1, Je);
            const T px = tail_fma((T)0.375, lds_ld<T>(n0) + lds_ld<T>(n1), (T)0.125 * (lds_ld<T>(f0) + lds_ld<T>(f1)));
            const unsigned a0 = tail_at<T>(C, base, I, J0) + Y, a1 = tail_at<T>(C, base, Ie, J0) + Y;
            const unsigned b0 = tail_at<T>(C, base, I, J1) + Y, b1 = tail_at<T>(C, base, Ie, J1) + Y;
            const T py = tail_fma((T)0.375, lds_ld<T>(a0) + lds_ld<T>(a1), (T)0.125 * (lds_ld<T>(b0) + lds_ld<T>(b1)));
            o[u][c].x = j < L.nx ? o[u][c].x + px : (T)0;
            o[u][c].y = i < L.ny ? o[u][c].y + py : (T)0;
        }
    }
    tail_put(L, pr, o);
}

// entries of the coarsest right-hand side in LDS: zero-padded to whole chunks
// of the dense solve's inner loop
constexpr int kDenseChunk = 256;
__host__ __device__ inline int tail_dense_pad(int nc) { return (nc + kDenseChunk - 1) / kDenseChunk * kDenseChunk; }

// LDS in bytes: [ E0 | spare word pair | per level below the top: E, R, V (the
// coarsest: E only) | rs ], E the iterate, R the right-hand side, V (eta_b,
// eta_p), rs the coarsest right-hand side in FP64.  E0 also takes the residual
// of whichever level is being restricted.
template <typename T>
__host__ __device__ inline size_t tail_area(int nx, int ny) { return (size_t)(ny + 2) * (nx + 2) * 2 * sizeof(T); }

template <typename T, int NT, int KP>
__device__ __forceinline__ void coarse_cycle_body(const CoarseArgs<T>& A) {
    using V2 = TailV2<T>;
    constexpr unsigned S = sizeof(V2);
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const unsigned lds0 = (unsigned)(uintptr_t)(TPH_LDS unsigned char*)smem_raw;
    const int nl = A.nl;
    const int tid = threadIdx.x;
    const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~63);       // first thread of this wave
    const bool gs = A.smoother == 1;
    const T om = A.omega;
    const V2 zero = {(T)0, (T)0};
    auto area = [&](int l) { return (unsigned)tail_area<T>(A.lv[l].nx, A.lv[l].ny); };
    auto owns = [&](int l) { return wave0 < (A.lv[l].nx >> 1) * A.lv[l].ny; };
    const unsigned spare = lds0 + area(0), base1 = spare + 16;
    unsigned rs = base1;
    for (int l = 1; l < nl; ++l) rs += (l < nl - 1 ? 3 : 1) * area(l);

    // The top level's pairs come straight from memory.  j0 is odd and entry
    // (i, 1) is aligned, so a pair's two columns are one aligned vector.
    auto load_top = [&](TailRaw<T> (&raw)[KP], TailPair<T> (&top)[KP]) {
        const int P = A.lv[0].pitch;
#pragma unroll
        for (int u = 0; u < KP; ++u) {
            tail_place(A.lv[0], lds0, spare, tid + u * NT, top[u]);
            const unsigned c = top[u].i * P + top[u].j0;
            TailRaw<T>& r = raw[u];
            r.p = *(const V2*)(A.ep[0] + c);
            r.pn = *(const V2*)(A.ep[0] + (c + P));
            r.pe = A.ep[0][c + 2];
            r.b = *(const V2*)(A.eb[0] + c);
            r.bs = *(const V2*)(A.eb[0] + (c - P));
            r.bw = A.eb[0][c - 1];
            r.rx = *(const V2*)(A.rx + c);
            r.ry = *(const V2*)(A.ry + c);
        }
    };
    // the pair this thread owns on a level below the top, whose arrays start at E
    auto load_pair = [&](int l, unsigned E, TailPair<T> (&pr)[1]) {
        const TailLevel<T>& L = A.lv[l];
        tail_place(L, E, spare, tid, pr[0]);
        const unsigned n = area(l), o = tail_at<T>(L, E, pr[0].i, pr[0].j0);
        const unsigned r0 = o + n, r1 = r0 + S - L.odd, v0 = r0 + n, v1 = v0 + S - L.odd;    // columns j0, j0 + 1
        constexpr unsigned Y = sizeof(T);
        const V2 e0 = lds_ld<V2>(v0), e1 = lds_ld<V2>(v1), q0 = lds_ld<V2>(r0), q1 = lds_ld<V2>(r1);
        TailRaw<T> r;
        r.p = V2{e0.y, e1.y};
        r.b = V2{e0.x, e1.x};
        r.pn = V2{lds_ld<T>(v0 + L.row + Y), lds_ld<T>(v1 + L.row + Y)};
        r.bs = V2{lds_ld<T>(v0 - L.row), lds_ld<T>(v1 - L.row)};
        r.pe = lds_ld<T>(v0 + S + Y);    // column j0 + 2: next in the odd half
        r.bw = lds_ld<T>(v1 - S);        // column j0 - 1: previous in the even half
        r.rx = V2{q0.x, q1.x};
        r.ry = V2{q0.y, q1.y};
        tail_finish(L, r, pr[0]);
    };
    // restrict the residual of level l in E0 to the next level: into its
    // right-hand side at R, or (the coarsest) the FP64 vector of unknowns
    auto restrict_from = [&](int l, unsigned R) {
        const TailLevel<T>&F = A.lv[l], &C = A.lv[l + 1];
        const int nc = C.nx * C.ny, nvx = C.ny * (C.nx - 1);
        // the x parts of all cells, then the y parts: independent work for every thread
        for (int t = tid; t < 2 * nc; t += NT) {
            const bool isx = t < nc;
            const int q = isx ? t : t - nc;
            const int r = small_div(q, C.rnx), I = 1 + r, J = 1 + q - r * C.nx;
            T v;
            if (isx) {
                if (J >= C.nx) continue;
                v = tail_restrict_x(F, lds0, C.ny, I, J);
            } else {
                if (I >= C.ny) continue;
                v = tail_restrict_y(F, lds0, C.nx, I, J);
            }
            if (l + 1 == nl - 1) lds_st<double>(rs + 8u * (isx ? (I - 1) * (C.nx - 1) + J - 1 : nvx + (I - 1) * C.nx + J - 1), (double)v);
            else lds_st<T>(tail_at<T>(C, R, I, J) + (isx ? 0u : (unsigned)sizeof(T)), v);
        }
        __syncthreads();
    };

    // ---- load: the top level's pairs; the viscosities of the levels between
    // it and the coarsest into LDS (one flat index, a batch of loads in flight
    // before the first is stored); every iterate zero
    TailPair<T> top[KP];
    TailRaw<T> raw[KP];
    load_top(raw, top);
    {
        int ntot = 0;
        for (int l = 1; l < nl - 1; ++l) ntot += (A.lv[l].ny + 2) * (A.lv[l].nx + 2);
        constexpr int KL = 4;
        for (int t0 = 0; t0 < ntot; t0 += KL * NT) {
            V2 v[KL];
            unsigned at[KL];
#pragma unroll
            for (int u = 0; u < KL; ++u) {
                int q = t0 + u * NT + tid, l = 1;
                unsigned E = base1;
                at[u] = 0;
                if (q >= ntot) continue;
                for (; q >= (A.lv[l].ny + 2) * (A.lv[l].nx + 2); ++l) {
                    q -= (A.lv[l].ny + 2) * (A.lv[l].nx + 2);
                    E += 3 * area(l);
                }
                const TailLevel<T>& L = A.lv[l];
                const int i = small_div(q, L.rp), j = q - i * (L.nx + 2);
                const unsigned c = i * L.pitch + j;
                v[u] = V2{A.eb[l][c], A.ep[l][c]};
                at[u] = tail_at<T>(L, E + 2 * area(l), i, j);
            }
#pragma unroll
            for (int u = 0; u < KL; ++u)
                if (at[u]) lds_st<V2>(at[u], v[u]);
        }
        for (unsigned a = lds0 + tid * S; a < lds0 + area(0) + S; a += NT * S) lds_st<V2>(a, zero);
        unsigned E = base1;
        for (int l = 1; l < nl; ++l) {
            for (unsigned a = E + tid * S; a < E + area(l); a += NT * S) lds_st<V2>(a, zero);
            E += 3 * area(l);
        }
        for (int t = A.nc + tid; t < tail_dense_pad(A.nc); t += NT) lds_st<double>(rs + 8 * t, 0.0);
    }
#pragma unroll
    for (int u = 0; u < KP; ++u) tail_finish(A.lv[0], raw[u], top[u]);
    __syncthreads();

    // ---- down, top level
    V2 o0[KP][2];
    tail_smooth<T, KP>(A.lv[0], om, top, A.nu_pre[0], gs, owns(0));
    {
        V2 t[KP][2];
        tail_residual<T, KP>(A.lv[0], top, o0, t);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < KP; ++u)
#pragma unroll
            for (int c = 0; c < 2; ++c) lds_st<V2>(top[u].a[c], t[u][c]);
        __syncthreads();
    }
    unsigned E = base1;                  // arrays of the current level below the top
    restrict_from(0, E + area(1));

    // Small coarsest systems: a lane's entries of the inverse go into
    // registers now, so their latency hides behind the levels in between.
    // Entries past the row's end repeat its last one; the zero padding of rs
    // takes them out.
    constexpr int kLanes = 16, KM = 8, NG = NT / kLanes, RM = 128 / NG;
    const int sub = tid & (kLanes - 1), grp = tid / kLanes;
    const bool minv_regs = A.nc <= kLanes * KM;
    double mv[RM][KM];
    if (minv_regs) {
        unsigned q[KM];
#pragma unroll
        for (int c = 0; c < KM; ++c) q[c] = min(sub + kLanes * c, A.nc - 1);
#pragma unroll
        for (int r = 0; r < RM; ++r) {
            const unsigned row = min(grp + r * NG, A.nc - 1) * A.nc;
#pragma unroll
            for (int c = 0; c < KM; ++c) mv[r][c] = A.Minv[row + q[c]];
        }
    }

    // ---- down, the levels below the top
    for (int l = 1; l < nl - 1; ++l) {
        const bool wave = owns(l);
        TailPair<T> pr[1];
        if (wave) load_pair(l, E, pr);
        tail_smooth<T, 1>(A.lv[l], om, pr, A.nu_pre[l], gs, wave);
        if (wave) {
            V2 o[1][2], t[1][2];
            tail_residual<T, 1>(A.lv[l], pr, o, t);
#pragma unroll
            for (int c = 0; c < 2; ++c)
                lds_st<V2>(pr[0].live ? pr[0].a[c] - E + lds0 : spare, t[0][c]);
        }
        __syncthreads();
        E += 3 * area(l);
        restrict_from(l, E + area(l + 1));
    }

    // the top level's pairs for the second leg, in flight from here on (up to two
    // per thread stay in registers instead)
    if constexpr (KP > 2) load_top(raw, top);

    // ---- coarsest: e = -(-L)^{-1} r in FP64; 16 lanes share a row of the
    // inverse, each summing every 16th entry
    {
        const TailLevel<T>&C = A.lv[nl - 1], &L0 = A.lv[0];
        const int nvx = C.ny * (C.nx - 1), n = A.nc;
        // the residuals in E0 are done with: the top level's walls, corners and ghosts back to zero
        for (int t = tid; t < L0.ny + 2; t += NT) {
            lds_st<V2>(tail_at<T>(L0, lds0, t, 0), zero);
            lds_st<V2>(tail_at<T>(L0, lds0, t, L0.nx + 1), zero);
        }
        for (int t = tid; t < L0.nx + 2; t += NT) {
            lds_st<V2>(lds0 + t * S, zero);
            lds_st<V2>(lds0 + (L0.ny + 1) * L0.row + t * S, zero);
        }
        auto put = [&](int m, double sv) {
            const T e = (T)(-sv);
            const bool isx = m < nvx;
            const int mm = isx ? m : m - nvx;
            const int r = small_div(mm, isx ? C.rnx1 : C.rnx), i = 1 + r, j = 1 + mm - r * (isx ? C.nx - 1 : C.nx);
            const unsigned a = tail_at<T>(C, E, i, j) + (isx ? 0u : (unsigned)sizeof(T));
            lds_st<T>(a, e);
            if (isx) {
                if (i == 1) lds_st<T>(a - C.row, C.mirS * e);
                if (i == C.ny) lds_st<T>(a + C.row, C.mirN * e);
            } else {
                const int east = (j & 1) ? (int)S - (int)C.odd : (int)C.odd, west = (j & 1) ? -(int)C.odd : (int)C.odd - (int)S;
                if (j == 1) lds_st<T>(a + west, C.mirW * e);
                if (j == C.nx) lds_st<T>(a + east, C.mirE * e);
            }
        };
        if (minv_regs) {
            double x[KM], mine = 0.0;
#pragma unroll
            for (int c = 0; c < KM; ++c) x[c] = lds_ld<double>(rs + 8 * (sub + kLanes * c));
#pragma unroll
            for (int r = 0; r < RM; ++r) {
                double sv = 0.0;
#pragma unroll
                for (int c = 0; c < KM; ++c) sv += mv[r][c] * x[c];
                sv = __shfl(row16_sum(sv), 0, kLanes);
                mine = sub == r ? sv : mine;         // lane r of the group keeps row r
            }
            const int m = grp + sub * NG;
            if (sub < RM && m < n) put(m, mine);
        } else {
            // two rows per group at a time, 16 entries of each in flight per lane;
            // loads past a row's end repeat its start and are left out
            constexpr int KD = kDenseChunk / kLanes;
            for (int m0 = grp; m0 < n; m0 += 2 * NG) {
                const int m1 = m0 + NG;
                const double* row0 = A.Minv + (unsigned)m0 * n;
                const double* row1 = A.Minv + (unsigned)min(m1, n - 1) * n;
                double s0 = 0.0, s1 = 0.0;
                for (int q0 = sub; q0 < n; q0 += kDenseChunk) {
                    double a0[KD], a1[KD];
#pragma unroll
                    for (int c = 0; c < KD; ++c) {
                        const unsigned q = q0 + kLanes * c < n ? q0 + kLanes * c : 0;
                        a0[c] = row0[q];
                        a1[c] = row1[q];
                    }
#pragma unroll
                    for (int c = 0; c < KD; ++c) {
                        const double x = lds_ld<double>(rs + 8 * (q0 + kLanes * c));
                        s0 += a0[c] * x;
                        s1 += a1[c] * x;
                    }
                }
                s0 = row16_sum(s0);
                s1 = row16_sum(s1);
                s1 = __shfl(s1, 0, kLanes);
                const int m = sub == 0 ? m0 : m1;
                if (sub < 2 && m < n) put(m, sub == 0 ? s0 : s1);
            }
        }
        __syncthreads();
    }

    // ---- up: prolong + correct, post-smooth
    for (int l = nl - 2; l >= 1; --l) {
        const bool wave = owns(l);
        const unsigned Ec = E;
        E -= 3 * area(l);
        TailPair<T> pr[1];
        if (wave) {
            load_pair(l, E, pr);
            V2 o[1][2] = {{lds_ld<V2>(pr[0].a[0]), lds_ld<V2>(pr[0].a[1])}};
            tail_correct<T, 1>(A.lv[l], A.lv[l + 1], Ec, pr, o);
        }
        __syncthreads();
        tail_smooth<T, 1>(A.lv[l], om, pr, A.nu_post[l], gs, wave);
    }
    tail_correct<T, KP>(A.lv[0], A.lv[1], E, top, o0);
    if constexpr (KP > 2) {
#pragma unroll
        for (int u = 0; u < KP; ++u) tail_finish(A.lv[0], raw[u], top[u]);
    }
    __syncthreads();
    tail_smooth<T, KP>(A.lv[0], om, top, A.nu_post[0], gs, owns(0));

    // ---- write the top-level correction (every entry: walls zero, ghosts mirrored)
    const TailLevel<T>& L0 = A.lv[0];
    for (int t = tid; t < (L0.ny + 2) * (L0.nx + 2); t += NT) {
        const int i = small_div(t, L0.rp), j = t - i * (L0.nx + 2);
        const V2 v = lds_ld<V2>(tail_at<T>(L0, lds0, i, j));
        A.ex[(unsigned)(i * L0.pitch + j)] = v.x;
        A.ey[(unsigned)(i * L0.pitch + j)] = v.y;
    }
}
#undef TPH_LDS

}  // namespace dev
}  // namespace tph
