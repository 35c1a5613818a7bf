// Marker <-> grid transfers and RK4 marker advection (Sec. "Interpolation
// Between Markers and Grid", Sec. "Advection of Lagrangian Markers",
// eq. rk4_method), behind the tph_markers_* entry points of tephra.h.
//
// Marker -> grid: markers are binned by the node-grid cell that contains them
// (the cell whose four corners are the nodes they weight) with a stable
// two-level partition written here (see k_keys); each cell then sums, in
// a fixed order, the weighted values and weights its markers give to its four
// corners, and each node adds the sums of its (up to) four cells in a fixed
// order.  Every sum has one writer and a fixed order, so results are bitwise
// reproducible.  Grid -> marker and RK4 are one thread per marker; all four
// RK4 stages run in registers, the velocity grids are read through the caches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <string>

#include "../../include/tephra.h"
#include "devmem.h"
#include "reduce.h"
#include "solver_internal.h"

struct tph_markers {
    int nx = 0, ny = 0;
    double lx = 0, ly = 0, dx = 0, dy = 0;
    int capacity = 0;
    hipStream_t st = nullptr;
    uint32_t* keys[2] = {nullptr, nullptr};
    int32_t* vals[2] = {nullptr, nullptr};
    int32_t* hist = nullptr;       // per (tile, digit) counts, then their scan over the tiles
    int32_t* total = nullptr;      // per digit
    int32_t* cstart = nullptr;     // per cell: first sorted position; one entry past the last cell
    const int32_t* order = nullptr;  // the sorted markers: one of vals
    // the current binning
    int kind = -1;
    int n = 0;
    const double* xm = nullptr;
    const double* ym = nullptr;
    tph::DeviceArena mem;          // device workspace (through the allocator current at creation)
};

namespace {

void tph_internal_set_error_m(const std::string& m) { tph_internal_set_error(m); }

// node grid of a kind: node (i, j) at (x0 + j dx, y0 + i dy), i in [imin, imax], j in [jmin, jmax]
struct NodeGrid {
    double x0, y0, dx, dy;
    int imin, imax, jmin, jmax;
    int pitch;                     // nx + 2: the caller's dense array layout
    double idx, idy;               // 1 / dx, 1 / dy (interpolation multiplies instead of dividing)
};

NodeGrid node_grid(const tph_markers* h, int kind) {
    NodeGrid q{};
    q.dx = h->dx;
    q.dy = h->dy;
    q.pitch = h->nx + 2;
    switch (kind) {
        case TPH_NODES_BASIC: q = {0.0, 0.0, h->dx, h->dy, 0, h->ny, 0, h->nx, h->nx + 2}; break;
        case TPH_NODES_CELL: q = {-0.5 * h->dx, -0.5 * h->dy, h->dx, h->dy, 1, h->ny, 1, h->nx, h->nx + 2}; break;
        case TPH_NODES_VX: q = {0.0, -0.5 * h->dy, h->dx, h->dy, 0, h->ny + 1, 0, h->nx, h->nx + 2}; break;
        default: q = {-0.5 * h->dx, 0.0, h->dx, h->dy, 0, h->ny, 0, h->nx + 1, h->nx + 2}; break;
    }
    q.idx = 1.0 / h->dx;
    q.idy = 1.0 / h->dy;
    return q;
}

// cells of the binning: lower-left node index (i, j) in [0, ny] x [0, nx] for both scatter kinds
__device__ __forceinline__ uint32_t cell_key(const NodeGrid& q, int nx, int ny, double x, double y) {
    int j = (int)floor((x - q.x0) / q.dx);
    int i = (int)floor((y - q.y0) / q.dy);
    j = j < 0 ? 0 : (j > nx ? nx : j);
    i = i < 0 ? 0 : (i > ny ? ny : i);
    return (uint32_t)(i * (nx + 1) + j);
}

// ---------------------------------------------------------------------------
// Binning: a stable partition of the marker indices by cell, in two levels.
// The cells (row-major) are cut into buckets of 2^s consecutive ones.
//   k_keys / k_digit_count: the markers of a tile (one workgroup, 16 waves of
//                   R rounds of 64 consecutive markers) per bucket -> hist
//   k_digit_offsets: per bucket, the scan over the tiles, and the total
//   k_digit_scatter: each marker to its bucket, in marker order
//   k_cell_sort:    one workgroup per bucket sorts its markers by cell within
//                   LDS counters and writes the first position of each cell
// A marker's rank among the earlier ones of its digit comes from ballots and
// from counts that each wave keeps in LDS, never from the order in which
// atomic operations arrive (the only atomics are integer counts, where the
// order does not matter): the order within a cell is that of the markers and
// results are bitwise reproducible.
// Bound by memory: per marker 16 B of position and a 4 B key written, read
// again, 6 B scattered and read, 4 B written.  A least-significant-digit
// sort over the whole key needs a pass of the pairs per 8 bits (three at
// 1024^2 cells) and another one for the ranges of the cells.
// ---------------------------------------------------------------------------
constexpr int kWaves = 16;

// entry i of an array below 4 GiB (at most 2^28 markers of up to 8 B): uniform base, 32-bit offset
template <typename T>
__device__ __forceinline__ const T& at32(const T* base, uint32_t i) {
    return *(const T*)((const char*)base + i * (uint32_t)sizeof(T));
}
template <typename T>
__device__ __forceinline__ T& at32(T* base, uint32_t i) {
    return *(T*)((char*)base + i * (uint32_t)sizeof(T));
}

constexpr int kSortRounds = 20;                  // k_cell_sort: markers of a bucket held at once, per lane
constexpr int kMaxShift = 11;                    // 2^11 cells a bucket: counts of 8 waves in 32 KB of LDS
constexpr int kMinShift = 5;
constexpr int kMaxBuckets = 2304;                // a 2048^2 grid in one pass (83 KB of LDS)
constexpr int kDigitBits = 12;                   // of a digit of a pass: below kMaxBuckets

// Lanes of `all` that hold the same digit (below 2^NB) as this one: four instructions a bit and no branch
// (a loop over the bits that are used took twice as long).
template <int NB>
__device__ __forceinline__ uint64_t digit_peers_bits(uint32_t d, uint64_t all) {
    uint32_t lo = (uint32_t)all, hi = (uint32_t)(all >> 32);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int32_t m = (int32_t)(d << (31 - b)) >> 31;
        const uint64_t bal = __ballot(m < 0);
        lo &= ~((uint32_t)bal ^ (uint32_t)m);
        hi &= ~((uint32_t)(bal >> 32) ^ (uint32_t)m);
    }
    return ((uint64_t)hi << 32) | lo;
}

// The same where few digits are likely.  Markers mostly come nearly in cell order, and then a wave holds a handful of digits: up to four are
// matched one by one, what is left bit by bit.
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, bool valid) {
    uint64_t rest = __ballot(valid), peers = 0;
    const uint64_t all = rest;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        if (!rest) return peers;
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, __builtin_ctzll(rest));
        const uint64_t same = __ballot(valid && d == d0);
        if (d == d0) peers = same;
        rest &= ~same;
    }
    if (!rest) return peers;
    return digit_peers_bits<kDigitBits>(d, all);
}

// Rank of this lane's item among the wave's earlier ones of its digit; cnt[d] (this wave's counts in LDS)
// is advanced.  FEW: a wave is likely to hold few digits.  Every lane of a group reads the count before the group's highest lane advances it: a
// wave's LDS operations complete in program order.
template <bool FEW>
__device__ __forceinline__ uint32_t wave_rank(uint32_t d, bool valid, int nbits, uint16_t* cnt) {
    const uint32_t base = cnt[d];
    const uint64_t peers = FEW          ? digit_peers(d, valid)
                           : nbits <= 9 ? digit_peers_bits<9>(d, __ballot(valid))
                                        : digit_peers_bits<kMaxShift>(d, __ballot(valid));
    const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
    const uint32_t all = (uint32_t)__popcll(peers);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (valid && below + 1 == all) cnt[d] = (uint16_t)(base + all);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return base + below;
}

// count of one digit per lane into hist (LDS): one addition per distinct digit while there are few
__device__ __forceinline__ void count_digit(uint32_t d, bool valid, int* hist) {
    const int lane = threadIdx.x & 63;
    uint64_t rest = __ballot(valid);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        if (!rest) return;
        const int first = __builtin_ctzll(rest);
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, first);
        const uint64_t same = __ballot(valid && d == d0);
        if (lane == first) atomicAdd(&hist[d0], __popcll(same));
        rest &= ~same;
    }
    if ((rest >> lane) & 1ull) atomicAdd(&hist[d], 1);
}

// exclusive scan over the workgroup's threads (NW waves) of one value each; ws: NW ints of LDS.  All call.
template <int NW>
__device__ __forceinline__ int block_exclusive(int v, int* ws) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int s = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(s, o);
        if (lane >= o) s += t;
    }
    if (lane == 63) ws[w] = s;
    __syncthreads();
    int before = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) before += q < w ? ws[q] : 0;
    __syncthreads();
    return before + s - v;
}

// Keys of the markers of a tile, and its counts of the first digit.  1024^2 cells, 16 markers each:
// 64 us, 5.2 TB/s (x, y and the keys: 335 MB).
template <int R>
__global__ __launch_bounds__(1024) void k_keys(NodeGrid q, int nx, int ny, int n, const double* __restrict__ xm,
                                               const double* __restrict__ ym, int shift, uint32_t mask, int ndig,
                                               uint32_t* __restrict__ keys, int32_t* __restrict__ hist) {
    __shared__ int cnt[kMaxBuckets];
    for (int d = threadIdx.x; d < ndig; d += 1024) cnt[d] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const long long m0 = ((long long)blockIdx.x * kWaves + w) * (R * 64) + lane;
    constexpr int U = R < 4 ? R : 4;             // loads of U rounds in flight
#pragma unroll
    for (int k0 = 0; k0 < R; k0 += U) {
        double x[U], y[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const long long m = m0 + (k0 + k) * 64;
            x[k] = m < n ? xm[m] : 0.0;
            y[k] = m < n ? ym[m] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const long long m = m0 + (k0 + k) * 64;
            const uint32_t key = cell_key(q, nx, ny, x[k], y[k]);
            if (m < n) keys[m] = key;
            count_digit((key >> shift) & mask, m < n, cnt);
        }
    }
    __syncthreads();
    for (int d = threadIdx.x; d < ndig; d += 1024) hist[(size_t)blockIdx.x * ndig + d] = cnt[d];
}

// the same counts of a further digit, from keys already in the order of the earlier one
template <int R>
__global__ __launch_bounds__(1024) void k_digit_count(const uint32_t* __restrict__ keys, int n, int shift,
                                                      uint32_t mask, int ndig, int32_t* __restrict__ hist) {
    __shared__ int cnt[kMaxBuckets];
    for (int d = threadIdx.x; d < ndig; d += 1024) cnt[d] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const long long m0 = ((long long)blockIdx.x * kWaves + w) * (R * 64) + lane;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const long long m = m0 + k * 64;
        const uint32_t key = m < n ? keys[m] : 0u;
        count_digit((key >> shift) & mask, m < n, cnt);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < ndig; d += 1024) hist[(size_t)blockIdx.x * ndig + d] = cnt[d];
}

// hist (tile-major: ndig counts per tile) -> per digit the exclusive scan over the tiles, in place, and its
// total.  16 digits per workgroup (64 B of a row), 64 runs of tiles.
__global__ __launch_bounds__(1024) void k_digit_offsets(int32_t* __restrict__ hist, int ntiles, int ndig,
                                                        int32_t* __restrict__ total) {
    __shared__ int part[64][17];
    const int c = threadIdx.x & 15, g = threadIdx.x >> 4;
    const int d = blockIdx.x * 16 + c;
    const bool live = d < ndig;
    const int per = (ntiles + 63) / 64;
    const int t0 = min(g * per, ntiles), t1 = min(t0 + per, ntiles);
    int s = 0;
    if (live) {
#pragma unroll 8
        for (int t = t0; t < t1; ++t) s += hist[(size_t)t * ndig + d];
    }
    part[g][c] = s;
    __syncthreads();
    for (int o = 1; o < 64; o <<= 1) {
        const int add = g >= o ? part[g - o][c] : 0;
        __syncthreads();
        part[g][c] += add;
        __syncthreads();
    }
    if (!live) return;
    int run = part[g][c] - s;
#pragma unroll 8
    for (int t = t0; t < t1; ++t) {
        const int v = hist[(size_t)t * ndig + d];
        hist[(size_t)t * ndig + d] = run;
        run += v;
    }
    if (g == 63) total[d] = part[g][c];
}

// Each marker to its digit's run: position = start of the digit + its earlier tiles + earlier waves + rank.
// K is uint16_t where this is the only pass (the bits below the digit are kept: all that k_cell_sort
// needs), uint32_t (whole keys) otherwise.  vin == nullptr: the markers are in their own order.
template <int R, typename K>
__global__ __launch_bounds__(1024, 8) void k_digit_scatter(const uint32_t* __restrict__ kin,
                                                        const int32_t* __restrict__ vin, int n, int shift,
                                                        uint32_t mask, int ndig,
                                                        const int32_t* __restrict__ hist,
                                                        const int32_t* __restrict__ total, K* __restrict__ kout,
                                                        int32_t* __restrict__ vout) {
    extern __shared__ int lds[];
    __shared__ int ws[kWaves];
    int* base = lds;                                                   // [ndig]
    uint16_t* wcnt = (uint16_t*)(lds + ndig);                          // [kWaves][ndig]
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t tile0 = blockIdx.x * (uint32_t)(kWaves * R * 64);
    const int left = min(n - (int)tile0, kWaves * R * 64);             // markers of the tile
    const int m0 = w * (R * 64) + lane;                                // within the tile
    uint32_t key[R], at[R];
#pragma unroll
    for (int k = 0; k < R; ++k) key[k] = m0 + k * 64 < left ? at32(kin + tile0, m0 + k * 64) : 0u;
    for (int d = threadIdx.x; d < ndig * (kWaves / 2); d += 1024) ((uint32_t*)wcnt)[d] = 0u;
    {
        constexpr int P = (kMaxBuckets + 1023) / 1024;
        int v[P], s = 0;
        const int d0 = threadIdx.x * P;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            v[p] = d0 + p < ndig ? total[d0 + p] : 0;
            s += v[p];
        }
        int run = block_exclusive<kWaves>(s, ws);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (d0 + p < ndig) base[d0 + p] = run + hist[(size_t)blockIdx.x * ndig + d0 + p];
            run += v[p];
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const uint32_t d = (key[k] >> shift) & mask;
        at[k] = wave_rank<true>(d, m0 + k * 64 < left, 0, wcnt + w * ndig);
        __builtin_amdgcn_sched_barrier(0);       // one round at a time: of their temporaries together more would spill
    }
    __syncthreads();
    for (int d = threadIdx.x; d < ndig; d += 1024) {
        uint32_t run = 0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) {
            const uint32_t c = wcnt[q * ndig + d];
            wcnt[q * ndig + d] = (uint16_t)run;                        // below 16 R 64 <= 16384
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int m = m0 + k * 64;
        asm("" : "+v"(key[k]));                  // the digit anew: 16 digits and addresses kept would spill (9 registers do)
        if (m < left) {
            const uint32_t d = (key[k] >> shift) & mask;
            const uint32_t pos = (uint32_t)base[d] + wcnt[w * ndig + d] + at[k];
            at32(kout, pos) = sizeof(K) == 2 ? (K)(key[k] & ((1u << shift) - 1u)) : (K)key[k];
            at32(vout, pos) = vin ? at32(vin + tile0, m) : (int32_t)(tile0 + m);
        }
    }
}

// first position whose key is at least `key`
__device__ __forceinline__ int lower_bound(const uint32_t* __restrict__ keys, int n, uint64_t key) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        if (keys[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Markers of one bucket (2^shift cells) to the order of the cells, and cstart of its cells.  A bucket of
// up to 10240 markers is ranked once, in registers; a longer one is counted first and goes in pieces.
// K as in k_digit_scatter: the bucket's run comes from the digit totals (uint16_t), or from a search in
// the sorted keys (uint32_t).  1024^2 cells, 16 markers each: 80 us with six waves a SIMD (eight: 91 us,
// with 20 registers spilled; five: 101 us).  At six the four-wave kernel still spills 12, the eight-wave one 4.
template <int NW, typename K>
__global__ __launch_bounds__(NW * 64, 6) void k_cell_sort(const K* __restrict__ kin, const int32_t* __restrict__ vin, int n,
                                                    int shift, int ncell, const int32_t* __restrict__ total,
                                                    int32_t* __restrict__ cstart, int32_t* __restrict__ order) {
    constexpr int R = kSortRounds;
    constexpr int NT = NW * 64;
    constexpr int P = (1 << kMaxShift) / NT;                           // at most that many cells a thread
    extern __shared__ int lds[];
    __shared__ int ws[NW];
    __shared__ int range[2];
    const int L = 1 << shift;
    int* base = lds;                                                   // [L]
    uint16_t* wcnt = (uint16_t*)(lds + L);                             // [NW][L]
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int c0 = (int)blockIdx.x << shift;
    const int nc = min(L, ncell - c0);
    int p0, cnt;
    if (sizeof(K) == 2) {
        int s = 0;
        for (int d = threadIdx.x; d < (int)blockIdx.x; d += NT) s += n ? total[d] : 0;
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (lane == 0) ws[w] = s;
        __syncthreads();
        p0 = 0;
#pragma unroll
        for (int q = 0; q < NW; ++q) p0 += ws[q];
        cnt = n ? total[blockIdx.x] : 0;
    } else {
        if (threadIdx.x < 2)
            range[threadIdx.x] = lower_bound((const uint32_t*)kin, n, ((uint64_t)blockIdx.x + threadIdx.x) << shift);
        __syncthreads();
        p0 = range[0];
        cnt = range[1] - p0;
    }
    const uint32_t mask = (uint32_t)L - 1u;
    const int per = (L + NT - 1) / NT;                                 // cells of a thread: consecutive ones
    const int mine = threadIdx.x * per;
    // positions of the cells from their counts; cstart
    auto place = [&](const int* tot) {
        int s = 0;
#pragma unroll
        for (int p = 0; p < P; ++p) s += tot[p];
        int run = p0 + block_exclusive<NW>(s, ws);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (p < per && mine + p < L) base[mine + p] = run;
            if (p < per && mine + p < nc) cstart[c0 + mine + p] = run;
            run += tot[p];
        }
    };
    if (threadIdx.x == 0 && c0 + nc == ncell) cstart[ncell] = n;
    const bool pieces = cnt > NW * R * 64;
    if (pieces) {
        for (int c = threadIdx.x; c < L; c += NT) base[c] = 0;
        __syncthreads();
        for (int t = threadIdx.x; t < cnt; t += NT) atomicAdd(&base[(uint32_t)kin[p0 + t] & mask], 1);
        __syncthreads();
        int tot[P];
#pragma unroll
        for (int p = 0; p < P; ++p) tot[p] = p < per && mine + p < L ? base[mine + p] : 0;
        place(tot);
    }
    int t0 = 0;
    do {
        const int left = min(cnt - t0, NW * R * 64);
        const int rounds = (left + NW * 64 - 1) / (NW * 64);   // at most R
        const int m0 = w * rounds * 64 + lane;                         // within the piece
        for (int c = threadIdx.x; c < L * (NW / 2); c += NT) ((uint32_t*)wcnt)[c] = 0u;
        uint32_t it[R];                                                // cell | rank within the wave << 16
#pragma unroll
        for (int k = 0; k < R; ++k) {
            it[k] = 0u;
            if (k < rounds && m0 + k * 64 < left) it[k] = (uint32_t)at32(kin + p0 + t0, m0 + k * 64) & mask;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < R; ++k) {
            if (k < rounds) it[k] |= wave_rank<false>(it[k], m0 + k * 64 < left, shift, wcnt + w * L) << 16;
            __builtin_amdgcn_sched_barrier(0);   // as in k_digit_scatter
        }
        __syncthreads();
        int tot[P];
        int own = mine;
        asm("" : "+v"(own));                     // no addresses kept over the pieces
#pragma unroll
        for (int p = 0; p < P; ++p) {
            uint32_t run = 0;
            if (p < per && own + p < L) {
#pragma unroll
                for (int q = 0; q < NW; ++q) {
                    const uint32_t c = wcnt[q * L + own + p];
                    wcnt[q * L + own + p] = (uint16_t)run;             // below 10240
                    run += c;
                }
            }
            tot[p] = (int)run;
        }
        if (!pieces) place(tot);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int t = m0 + k * 64;
            asm("" : "+v"(it[k]));                                     // as in k_digit_scatter
            if (k < rounds && t < left) {
                const uint32_t c = it[k] & 0xffffu;
                at32(order, (uint32_t)base[c] + wcnt[w * L + c] + (it[k] >> 16)) = at32(vin + p0 + t0, t);
            }
        }
        t0 += left;
        if (t0 < cnt) {                                                // the same for every thread
            __syncthreads();
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (p < per && mine + p < L) base[mine + p] += tot[p];
        }
    } while (t0 < cnt);
}

// Factors rx, ry of a marker's weights in its cell: the quotients of the direct formulas.  Those by the
// spacing are had from its reciprocal and two corrections (a third of a division's operations); the
// cell column by a product, unless that is so close to a column's edge, or so far out, that the division
// that gave the key might say otherwise: then (false) everything is to be divided.
__device__ __forceinline__ double by_spacing(double a, double h, double ih) {
    double v = a * ih;
    v = __builtin_fma(__builtin_fma(-h, v, a), ih, v);
    return __builtin_fma(__builtin_fma(-h, v, a), ih, v);
}

__device__ __forceinline__ bool factors(const NodeGrid& q, int nx, double x, double y, double yi, double& rx,
                                        double& ry) {
    const double t = (x - q.x0) * q.idx;
    int j = (int)floor(t);
    j = j < 0 ? 0 : (j > nx ? nx : j);
    rx = by_spacing(x - (q.x0 + j * q.dx), q.dx, q.idx);
    ry = by_spacing(y - yi, q.dy, q.idy);
    return fabs(t - rint(t)) > 0x1p-20 && fabs(y - yi) < 0x1p40 * q.dy;  // false for NaN
}

__device__ __forceinline__ void divided_factors(const NodeGrid& q, int nx, double x, double y, double yi, double& rx,
                                                double& ry) {
    int j = (int)floor((x - q.x0) / q.dx);
    j = j < 0 ? 0 : (j > nx ? nx : j);
    rx = (x - (q.x0 + j * q.dx)) / q.dx;
    ry = (y - yi) / q.dy;
}

// ---------------------------------------------------------------------------
// Averages on the nodes from the sorted markers.  Per cell, in sorted order:
// sums of w phi and w for its four corners; node (i, j) = corner (1,1) of
// cell (i-1, j-1), (1,0) of (i-1, j), (0,1) of (i, j-1), (0,0) of (i, j), in
// that order.  A wave takes 64 neighbouring cells of R rows, 16 at a time:
// their markers are one run of the sorted order.
//   Its markers, one per lane, are gathered, their positions become the two
// factors of the weights, and both go to LDS with phi; then four lanes walk
// each cell's markers, one corner each (5 operations a marker instead of 16
// on a quarter of the lanes).  The gathers of the next 16 cells are in flight
// meanwhile.  Slots are padded by one per 16: neighbouring cells start
// about 16 markers apart, which would otherwise put their reads on the same
// LDS banks.
//   The sums of a row go through LDS once, to the lanes of the nodes; the row
// above's are kept in registers, those of the wave before come through
// LDS.  Lane 0 of a wave is a cell for the node of lane 1 only, and a
// workgroup's first cell row is the last one of the workgroup above.
// Bound by the gathers (28 B a marker: 95 us at the rate of a copy at 1024^2 cells of 16 markers; 146 us,
// from 173 with a pass over partial sums in memory) and by the walk's operations.
// ---------------------------------------------------------------------------
constexpr int kNodeWaves = 4;
// Runs (of 16 cells) beyond this many markers go cell by cell, 16 lanes a corner.  A lane a corner walks one marker
// after the other at some 150 cycles each, and in a crowd, where a staged piece covers a cell or less, the other 60
// wait: 4.2 M markers on 1024^2 cells, gathered in a tenth of the rows and columns (400 a cell), 4400 -> 380 us of
// this kernel.  The line lies where both take the same: at 16 a cell (runs of 256) walking takes 196 us a call, cell
// by cell 215; at 33 a cell 259 and 248.
constexpr int kCrowd = 512;
// sum over the sixteen lanes that share lane & 3, in all of them
__device__ __forceinline__ double sixteen_sum(double v) {
    v = tph::wave_add_rows(tph::wave_add_halves(v));
    v += tph::row16_rotate<0x128>(v);
    return v + tph::row16_rotate<0x124>(v);
}
__device__ __forceinline__ int stage_slot(int t) { return t + (t >> 4); }

// every node of the range, where there are no markers
__global__ __launch_bounds__(256) void k_fill_nodes(NodeGrid q, double fill, double* __restrict__ grid) {
    const int j = q.jmin + (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (j <= q.jmax) grid[(size_t)(q.imin + (int)blockIdx.y) * q.pitch + j] = fill;
}

// H: markers a lane holds, 64 H the piece that is staged at once
template <int R, int H>
__global__ __launch_bounds__(kNodeWaves * 64) void k_nodes(NodeGrid q, int nx, int ny,
                                                           const int32_t* __restrict__ cstart,
                                                           const int32_t* __restrict__ order,
                                                           const double* __restrict__ xm,
                                                           const double* __restrict__ ym,
                                                           const double* __restrict__ phi, double fill,
                                                           double* __restrict__ grid) {
    constexpr int kChunk = H * 64;
    constexpr int kSlots = kChunk + kChunk / 16 + 4;                   // an even number, past the walk's last read
    __shared__ double stage[kNodeWaves][3 * kSlots];
    __shared__ double2 corners[kNodeWaves][4][64];                     // (sum w phi, sum w) of a row's cells
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double* sx = stage[w];
    double* sy = sx + kSlots;
    double* sf = sy + kSlots;
    const int jl = (int)blockIdx.x * 63 - 1;                           // cell column of lane 0
    const int j = jl + lane;
    const int i0 = (int)blockIdx.y * (kNodeWaves * R - 1) - 1 + w * R; // first cell row of the wave
    const bool col = j >= 0 && j <= nx;
    const int corner = lane & 3;
    // weight of this lane's corner: (ax + bx rx)(ay + by ry), that is 1 - r or r
    const double ax = corner & 1 ? 0.0 : 1.0, bx = corner & 1 ? 1.0 : -1.0;
    const double ay = corner & 2 ? 0.0 : 1.0, by = corner & 2 ? 1.0 : -1.0;
    // cell ranges of a row; columns and rows outside are empty, at the end or the start of their neighbours'
    auto range = [&](int i, int& b, int& e) {
        const bool live = i >= 0 && i <= ny;
        const uint32_t c = (uint32_t)i * (uint32_t)(nx + 1);
        b = live ? at32(cstart, c + (uint32_t)min(max(j, 0), nx + 1)) : 0;
        e = live ? at32(cstart, c + (uint32_t)min(max(j + 1, 0), nx + 1)) : 0;
    };
    int b, e, b1, e1;                                                  // this row's, the next one's
    int m[H];
    double vx[H], vy[H], vf[H];
    // straight-line code: with a branch around a round, each would wait for the one before.  A lane past the
    // run takes its last marker (some marker, if the run is empty).
    auto indices = [&](int P0, int P1) {
#pragma unroll
        for (int k = 0; k < H; ++k) m[k] = at32(order, min(P0 + k * 64 + lane, max(P1 - 1, 0)));
    };
    auto gather = [&]() {
#pragma unroll
        for (int k = 0; k < H; ++k) {
            vx[k] = at32(xm, m[k]);
            vy[k] = at32(ym, m[k]);
            vf[k] = at32(phi, m[k]);
        }
    };
    auto to_lds = [&](double yi) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        double rx[H], ry[H];
        bool unsure = false;
#pragma unroll
        for (int k = 0; k < H; ++k) unsure |= !factors(q, nx, vx[k], vy[k], yi, rx[k], ry[k]);
        if (unsure) {
#pragma unroll
            for (int k = 0; k < H; ++k) divided_factors(q, nx, vx[k], vy[k], yi, rx[k], ry[k]);
        }
#pragma unroll
        for (int k = 0; k < H; ++k) {
            const int t = stage_slot(lane + k * 64);
            sx[t] = rx[k];
            sy[t] = ry[k];
            sf[t] = vf[k];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    double num, den;
    auto add = [&](double rx, double ry, double f) {
        const double wt = __builtin_fma(bx, rx, ax) * __builtin_fma(by, ry, ay);
        num = __builtin_fma(wt, f, num);
        den += wt;
    };
    // positions [u, ue) of the run from P0, two at a time, the next two's reads ahead of these two's sums
    auto walk = [&](int u, int ue, int P0) {
        if (u >= ue) return;
        int t = stage_slot(u - P0), t1 = stage_slot(u + 1 - P0);
        double rx = sx[t], ry = sy[t], f = sf[t], rx1 = sx[t1], ry1 = sy[t1], f1 = sf[t1];
        while (u + 1 < ue) {
            u += 2;
            t = stage_slot(u - P0);
            t1 = stage_slot(u + 1 - P0);
            const double nx0 = sx[t], ny0 = sy[t], nf0 = sf[t], nx1 = sx[t1], ny1 = sy[t1], nf1 = sf[t1];
            add(rx, ry, f);
            add(rx1, ry1, f1);
            rx = nx0;
            ry = ny0;
            f = nf0;
            rx1 = nx1;
            ry1 = ny1;
            f1 = nf1;
        }
        if (u < ue) add(rx, ry, f);
    };
    // A crowded run: one cell after the other, each by all lanes.  Sixteen lanes a corner take a cell's markers in
    // turn (by their rank in the cell, whatever the pieces) and their sums are added in the tree of halving
    // distances; lanes of cell c of the sixteen end with its sums.
    auto walk_crowded = [&](int g, int P0, int P1, double yi) {
        int c = 0, cs = P0, ce = __builtin_amdgcn_readlane(e, g * 16);
        double own_num = 0.0, own_den = 0.0;
        indices(P0 + kChunk, P1);
#pragma unroll 1
        for (int p = P0;; p += kChunk) {
            gather();
            indices(p + 2 * kChunk, P1);
            const int pe = min(p + kChunk, P1);
#pragma unroll 1
            for (;;) {
                const int u = max(cs, p);
                for (int t = u + (((lane >> 2) - (u - cs)) & 15); t < min(ce, pe); t += 16) {
                    const int q = stage_slot(t - p);
                    add(sx[q], sy[q], sf[q]);
                }
                if (ce > pe || c == 15) break;
                num = sixteen_sum(num);
                den = sixteen_sum(den);
                own_num = lane >> 2 == c ? num : own_num;
                own_den = lane >> 2 == c ? den : own_den;
                num = den = 0.0;
                ++c;
                cs = ce;
                ce = __builtin_amdgcn_readlane(e, g * 16 + c);
            }
            if (p + kChunk >= P1) break;
            to_lds(yi);
        }
        num = sixteen_sum(num);
        den = sixteen_sum(den);
        num = lane >> 2 == 15 ? num : own_num;
        den = lane >> 2 == 15 ? den : own_den;
    };
    auto run_of = [&](int g, int bb, int ee, int& P0, int& P1) {
        P0 = __builtin_amdgcn_readlane(bb, g * 16);
        P1 = __builtin_amdgcn_readlane(ee, g * 16 + 15);
    };
    double2 up[2], top[2];                                             // corners 3, 2 of the row above; 1, 0 of the first row
    auto node = [&](int i, double2 c1, double2 c0) {
        double n = up[0].x, d = up[0].y;
        n += up[1].x;
        d += up[1].y;
        n += c1.x;
        d += c1.y;
        n += c0.x;
        d += c0.y;
        if (lane > 0 && i >= q.imin && i <= q.imax && j >= q.jmin && j <= q.jmax)
            grid[(size_t)i * q.pitch + j] = d > 0.0 ? n / d : fill;
    };
    range(i0, b, e);
    if (R > 1) range(i0 + 1, b1, e1);
    int P0, P1;
    run_of(0, b, e, P0, P1);
    indices(P0, P1);
    gather();
    int N0, N1;
    run_of(1, b, e, N0, N1);
    indices(N0, N1);
#pragma unroll 1
    for (int gg = 0; gg < 4 * R; ++gg) {
        const int g = gg & 3, i = i0 + (gg >> 2);
        const double yi = q.y0 + i * q.dy;
        const int cb = __shfl(b, g * 16 + (lane >> 2)), ce = __shfl(e, g * 16 + (lane >> 2));
        // the run after the next one
        int M0 = 0, M1 = 0;
        if (g < 2) run_of(g + 2, b, e, M0, M1);
        else if (gg + 2 < 4 * R) run_of(g - 2, b1, e1, M0, M1);
        num = den = 0.0;
        to_lds(yi);
        if (P1 - P0 <= kChunk) {
            gather();
            indices(M0, M1);
            walk(cb, ce, P0);
        } else {
            if (P1 - P0 > kCrowd) {
                walk_crowded(g, P0, P1, yi);
            } else {
                walk(cb, min(ce, P0 + kChunk), P0);
                for (int p = P0 + kChunk; p < P1; p += kChunk) {
                    const int pe = min(p + kChunk, P1);
                    indices(p, pe);
                    gather();
                    to_lds(yi);
                    walk(max(cb, p), min(ce, pe), p);
                }
            }
            indices(N0, N1);
            gather();
            indices(M0, M1);
        }
        P0 = N0;
        P1 = N1;
        N0 = M0;
        N1 = M1;
        corners[w][corner][g * 16 + (lane >> 2)] = make_double2(num, den);
        if (g == 3) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const int l1 = max(lane - 1, 0);
            const double2 c1 = corners[w][1][l1], c0 = corners[w][0][lane];
            if (gg == 3) {
                top[0] = c1;
                top[1] = c0;
            } else {
                node(i, c1, c0);
            }
            up[0] = corners[w][3][l1];
            up[1] = corners[w][2][lane];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            b = b1;
            e = e1;
            if (gg + 4 < 4 * R) range(i + 2, b1, e1);
        }
    }
    double2* mine = (double2*)stage[w];
    mine[lane] = up[0];
    mine[64 + lane] = up[1];
    __syncthreads();
    if (w == 0) return;                                                // its first row's nodes are the workgroup above's
    const double2* before = (const double2*)stage[w - 1];
    up[0] = before[lane];
    up[1] = before[64 + lane];
    node(i0, top[0], top[1]);
}

// two neighbouring entries of a row, wherever the pair starts
typedef double Pair __attribute__((ext_vector_type(2), aligned(8)));

// where a marker is in a node grid: the first node of its cell, and its parts of the cell
struct Place {
    uint32_t at;
    double rx, ry;
};

// (the cell found by a multiplication may differ from the divided one for a
// marker on a cell edge; both cells give the same value there).  The parts of the
// cell come from the unrounded product, which can lie below the node line that
// the rounded one was taken to, and the cell is kept in the node range: both are
// clamped to [0, 1].
__device__ __forceinline__ Place place(const NodeGrid& q, double x, double y) {
    const double ax = x - q.x0, ay = y - q.y0;
    int j = (int)floor(ax * q.idx), i = (int)floor(ay * q.idy);
    j = j < q.jmin ? q.jmin : (j > q.jmax - 1 ? q.jmax - 1 : j);
    i = i < q.imin ? q.imin : (i > q.imax - 1 ? q.imax - 1 : i);
    double rx = __builtin_fma(ax, q.idx, -(double)j), ry = __builtin_fma(ay, q.idy, -(double)i);
    rx = rx < 0.0 ? 0.0 : (rx > 1.0 ? 1.0 : rx);
    ry = ry < 0.0 ? 0.0 : (ry > 1.0 ? 1.0 : ry);
    return {(uint32_t)(i * q.pitch + j), rx, ry};
}

// The same in fewer operations and with a branch: a cell of the node range needs no clamp of its numbers, and its
// parts only one from below; a wave with a marker outside, or at no position, takes the long way.
__device__ __forceinline__ Place place_short(const NodeGrid& q, double x, double y) {
    const double ax = x - q.x0, ay = y - q.y0;
    const double fx = floor(ax * q.idx), fy = floor(ay * q.idy);
    const int j = (int)fx, i = (int)fy;
    const double any = fx + fy;                  // NaN if one is
    // one condition, not a chain of branches
    if (((unsigned)(j - q.jmin) >= (unsigned)(q.jmax - q.jmin)) | ((unsigned)(i - q.imin) >= (unsigned)(q.imax - q.imin)) |
        (any != any))
        return place(q, x, y);
    return {(uint32_t)(i * q.pitch + j), __builtin_fmax(__builtin_fma(ax, q.idx, -fx), 0.0),
            __builtin_fmax(__builtin_fma(ay, q.idy, -fy), 0.0)};
}

// the four nodes of a cell: a row's two in one load
struct Cell {
    Pair a, b;
};
__device__ __forceinline__ Cell cell_of(const NodeGrid& q, const double* __restrict__ grid, uint32_t at) {
    const double* g0 = grid + at;
    return {*(const Pair*)g0, *(const Pair*)(g0 + q.pitch)};
}

// The sum of four weighted nodes.  The weights add up to one and each product rounds by itself, so the error is
// relative to the result whatever the ratio of the nodes, and a marker on a node gets its value.  Three
// differences, a.x + r (a.y - a.x), are four operations fewer and round at the largest node: 2e-10 of the result
// at a ratio of 1e6, where this gives 4e-16.  The fused operations are spelled out: their order decides the bits.
__device__ __forceinline__ double interp(const Cell& c, const Place& m) {
    const double rx = m.rx, ry = m.ry;
    const double sx = 1.0 - rx, sy = 1.0 - ry;
    return __builtin_fma(rx * ry, c.b.y, __builtin_fma(sx * ry, c.b.x, __builtin_fma(sx * sy, c.a.x, rx * sy * c.a.y)));
}

__global__ __launch_bounds__(256) void k_from_grid(NodeGrid q, int n, const double* __restrict__ xm,
                                                   const double* __restrict__ ym, const double* __restrict__ grid,
                                                   double* __restrict__ out) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    const Place at = place(q, xm[m], ym[m]);
    out[m] = interp(cell_of(q, grid, at.at), at);
}

// KEEP, for many markers: bound by the gathers of the velocity (16 loads a marker).  A stage moves a marker by a
// fraction of a cell in a usual step: most lanes are still in the cell of the stage before and keep its nodes.
// Otherwise, for few: bound by the latency of four gathers in a row, with no branch between them.  500, 65 000,
// 130 000, 270 000 and 2.9 M markers: 3.1, 4.1, 4.7, 7.1 and 37.0 us with, 2.6, 3.7, 4.6, 7.4 and 43.1 without,
// sorted by cell.  In random order keeping pays earlier: whole calls of 32 000, 65 000, 100 000 and 200 000 markers
// take 19.4, 19.5, 20.0 and 23.3 us with, 19.4, 20.2, 23.3 and 31.0 without; the line lies between.
template <bool KEEP>
__global__ __launch_bounds__(256) void k_rk4(NodeGrid qx, NodeGrid qy, double lx, double ly, int n,
                                             double* __restrict__ xm, double* __restrict__ ym,
                                             const double* __restrict__ vx, const double* __restrict__ vy, double dt) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    auto clampx = [&](double v) { return v < 0.0 ? 0.0 : (v > lx ? lx : v); };
    auto clampy = [&](double v) { return v < 0.0 ? 0.0 : (v > ly ? ly : v); };
    auto at = [](const NodeGrid& q, double u, double v) { return KEEP ? place_short(q, u, v) : place(q, u, v); };
    const double x = xm[m], y = ym[m];
    Place px = at(qx, x, y), py = at(qy, x, y);
    Cell cx = cell_of(qx, vx, px.at), cy = cell_of(qy, vy, py.at);
    // velocity at (u, v); both components' nodes together, so that their latencies overlap
    auto velocity = [&](double u, double v, double& kx, double& ky) {
        const Place nx = at(qx, u, v), ny = at(qy, u, v);
        if (!KEEP || nx.at != px.at || ny.at != py.at) {
            cx = cell_of(qx, vx, nx.at);
            cy = cell_of(qy, vy, ny.at);
        }
        px = nx;
        py = ny;
        kx = interp(cx, nx);
        ky = interp(cy, ny);
    };
    const double k1x = interp(cx, px), k1y = interp(cy, py);
    double k2x, k2y, k3x, k3y, k4x, k4y;
    double sx = clampx(x + 0.5 * dt * k1x), sy = clampy(y + 0.5 * dt * k1y);
    velocity(sx, sy, k2x, k2y);
    sx = clampx(x + 0.5 * dt * k2x);
    sy = clampy(y + 0.5 * dt * k2y);
    velocity(sx, sy, k3x, k3y);
    sx = clampx(x + dt * k3x);
    sy = clampy(y + dt * k3y);
    velocity(sx, sy, k4x, k4y);
    xm[m] = clampx(x + dt / 6.0 * (k1x + 2.0 * k2x + 2.0 * k3x + k4x));
    ym[m] = clampy(y + dt / 6.0 * (k1y + 2.0 * k2y + 2.0 * k3y + k4y));
}

constexpr int kFewMarkers = 60000;

inline unsigned blocks(long long n) { return (unsigned)((n + 255) / 256); }

#define M_HIP(call)                                                                                  \
    do {                                                                                             \
        hipError_t e_ = (call);                                                                      \
        if (e_ != hipSuccess) {                                                                      \
            tph_internal_set_error_m(std::string("HIP error in ") + #call + ": " + hipGetErrorString(e_)); \
            return TPH_ERR_HIP;                                                                      \
        }                                                                                            \
    } while (0)

constexpr int kMaxMarkers = 1 << 28;

// One cell row a wave while a small grid leaves the chip idle, two on larger ones: an eighth of the rows is then
// done twice (four rows: 172 us instead of 157 at 1024^2, with too few workgroups for an even last wave).
// A binning and six fields of 9 markers a cell, one row a wave and two: 300^2 cells 138 and 156 us, 500^2 223 and
// 227, 547^2 240 and 226, 1024^2 577 and 538; with 4 a cell both meet near 700^2, with 16 near 400^2.
constexpr long long kRowCells = 300000;

// How the bits of a key are divided: the lowest `shift` within a bucket, the rest in one pass or two.
// One pass as long as its counts fit in LDS; two of about equal width beyond 2304 buckets of 2048 cells
// (grids above 4.7 M cells).
struct BinPlan {
    int shift = 0, npass = 1;
    int buckets = 0;               // of 2^shift cells
    int bits[2] = {0, 0};          // of each pass
    int ndig[2] = {0, 0};
    int most() const { return std::max(ndig[0], ndig[1]); }
};

BinPlan bin_plan(const tph_markers* h) {
    const int ncell = (h->nx + 1) * (h->ny + 1);
    BinPlan p;
    // as many buckets as one pass can tell apart: with 512 cells each at 1024^2 x 16 markers k_cell_sort takes 80 us, with
    // 1024 cells some 40 us more, and the other kernels 8 us less
    p.shift = kMinShift;
    auto count = [&] { return (int)(((long long)ncell + (1ll << p.shift) - 1) >> p.shift); };
    while (p.shift < kMaxShift && count() > kMaxBuckets) ++p.shift;
    p.buckets = count();
    int nb = 1;
    while ((1ll << nb) < p.buckets) ++nb;
    if (p.buckets <= kMaxBuckets) {
        p.bits[0] = nb;
        p.ndig[0] = p.buckets;
    } else {
        p.npass = 2;
        p.bits[0] = nb / 2;
        p.bits[1] = nb - nb / 2;
        for (int k = 0; k < 2; ++k) p.ndig[k] = 1 << p.bits[k];
    }
    return p;
}

// Rounds of a tile (kWaves * 64 markers each): few for few markers, so that there is a workgroup for
// every CU; many for many, which keeps the table of counts (ndig per tile) small against them.
int tile_rounds(long long n) { return n <= (1 << 18) ? 1 : n <= (1 << 22) ? 4 : 16; }
long long tiles_of(long long n) {
    const long long t = (long long)tile_rounds(n) * kWaves * 64;
    return (n + t - 1) / t;
}

// LDS of a scatter pass with that many digits
constexpr size_t scatter_lds(int ndig) { return (size_t)ndig * (sizeof(int) + kWaves * sizeof(uint16_t)); }

template <int R>
hipError_t launch_pass(tph_markers* h, const BinPlan& p, const NodeGrid& q, int pass) {
    const int ntiles = (int)tiles_of(h->n), n = h->n;
    const int shift = p.shift + (pass ? p.bits[0] : 0), bits = p.bits[pass], ndig = p.ndig[pass];
    const uint32_t mask = (1u << bits) - 1u;
    const size_t lds = scatter_lds(ndig);
    if (pass == 0)
        hipLaunchKernelGGL((k_keys<R>), dim3(ntiles), dim3(1024), 0, h->st, q, h->nx, h->ny, n, h->xm, h->ym, shift, mask,
                           ndig, h->keys[0], h->hist);
    else
        hipLaunchKernelGGL((k_digit_count<R>), dim3(ntiles), dim3(1024), 0, h->st, h->keys[pass & 1], n, shift, mask, ndig,
                           h->hist);
    hipLaunchKernelGGL(k_digit_offsets, dim3((unsigned)((ndig + 15) / 16)), dim3(1024), 0, h->st, h->hist, ntiles, ndig,
                       h->total);
    const int32_t* vin = pass ? h->vals[(pass + 1) & 1] : nullptr;
    if (p.npass == 1)
        hipLaunchKernelGGL((k_digit_scatter<R, uint16_t>), dim3(ntiles), dim3(1024), lds, h->st, h->keys[0], vin, n, shift,
                           mask, ndig, h->hist, h->total, (uint16_t*)h->keys[1], h->vals[0]);
    else
        hipLaunchKernelGGL((k_digit_scatter<R, uint32_t>), dim3(ntiles), dim3(1024), lds, h->st, h->keys[pass & 1], vin, n,
                           shift, mask, ndig, h->hist, h->total, h->keys[1 - (pass & 1)], h->vals[pass & 1]);
    return hipGetLastError();
}

// The scatter's LDS exceeds 64 KB with more than 1820 digits.  The limit belongs to the function, not to a handle:
// every handle asks for the most that any of them can need, so that none lowers it under another.
hipError_t grant_lds() {
    const void* f[] = {(const void*)&k_digit_scatter<1, uint16_t>, (const void*)&k_digit_scatter<4, uint16_t>,
                       (const void*)&k_digit_scatter<16, uint16_t>};
    hipError_t e = hipSuccess;
    for (const void* k : f)
        if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)scatter_lds(kMaxBuckets));
    return e;
}

}  // namespace

extern "C" {

tph_status tph_markers_create(int32_t nx, int32_t ny, double lx, double ly, int32_t capacity, void* hip_stream,
                              tph_markers** out) {
    tph_internal_set_error_m("");
    if (!out) {
        tph_internal_set_error_m("out is NULL");
        return TPH_ERR_INVALID;
    }
    *out = nullptr;
    if (nx < 1 || ny < 1 || (int64_t)(nx + 2) * (ny + 2) > (int64_t)1 << 30 || !(lx > 0) || !(ly > 0) ||
        !std::isfinite(lx) || !std::isfinite(ly) || capacity < 1 || capacity > kMaxMarkers) {
        tph_internal_set_error_m("need nx, ny >= 1 (grid at most 2^30 entries), positive finite lx, ly and capacity "
                                 "in [1, 2^28]");
        return TPH_ERR_INVALID;
    }
    tph_markers* h = new tph_markers();
    h->nx = nx;
    h->ny = ny;
    h->lx = lx;
    h->ly = ly;
    h->dx = lx / nx;
    h->dy = ly / ny;
    h->capacity = capacity;
    h->st = (hipStream_t)hip_stream;
    h->mem.a = tph::default_allocator();
    const size_t ncell = (size_t)(nx + 1) * (ny + 1);
    std::string what;
    hipError_t e = hipSuccess;
    auto get = [&](void** p, size_t bytes) {
        if (e == hipSuccess) e = h->mem.alloc(p, bytes, &what);
    };
    for (int k = 0; k < 2; ++k) {
        get((void**)&h->keys[k], (size_t)capacity * sizeof(uint32_t));
        get((void**)&h->vals[k], (size_t)capacity * sizeof(int32_t));
    }
    get((void**)&h->cstart, (ncell + 1) * sizeof(int32_t));
    const BinPlan p = bin_plan(h);
    long long ntiles = 1;          // the most over the counts up to capacity
    for (long long n : {1ll << 18, 1ll << 22, (long long)kMaxMarkers})
        ntiles = std::max(ntiles, tiles_of(std::min<long long>(n, capacity)));
    get((void**)&h->hist, (size_t)ntiles * p.most() * sizeof(int32_t));
    get((void**)&h->total, (size_t)p.most() * sizeof(int32_t));
    if (e == hipSuccess) {
        e = grant_lds();
        what = "LDS for the binning kernels";
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        tph_markers_destroy(h);
        tph_internal_set_error_m("marker workspace: " + what);
        return e == hipErrorOutOfMemory ? TPH_ERR_OOM : TPH_ERR_HIP;
    }
    *out = h;
    return TPH_OK;
}

void tph_markers_destroy(tph_markers* h) {
    if (!h) return;
    if (h->st) (void)hipStreamSynchronize(h->st);
    h->mem.release_all();
    delete h;
}

tph_status tph_markers_bin(tph_markers* h, int32_t kind, int32_t n, const double* xm, const double* ym) {
    tph_internal_set_error_m("");
    if (!h || (n > 0 && (!xm || !ym))) {
        tph_internal_set_error_m("handle, xm and ym are required");
        return TPH_ERR_INVALID;
    }
    if (kind != TPH_NODES_BASIC && kind != TPH_NODES_CELL) {
        tph_internal_set_error_m("marker -> grid transfers go to TPH_NODES_BASIC or TPH_NODES_CELL");
        return TPH_ERR_INVALID;
    }
    if (n < 0 || n > h->capacity) {
        tph_internal_set_error_m("n must be in [0, capacity]");
        return TPH_ERR_INVALID;
    }
    const NodeGrid q = node_grid(h, kind);
    h->kind = -1;                  // no binning until all of its launches went through
    h->n = n;
    h->xm = xm;
    h->ym = ym;
    const BinPlan p = bin_plan(h);
    if (n > 0)
        for (int pass = 0; pass < p.npass; ++pass) {
            const int R = tile_rounds(n);
            M_HIP(R == 1 ? launch_pass<1>(h, p, q, pass) : R == 4 ? launch_pass<4>(h, p, q, pass)
                                                                  : launch_pass<16>(h, p, q, pass));
        }
    // one pass: from (keys[1], vals[0]) to vals[1]; two: from (keys[0], vals[1]) to vals[0]
    const int ncell = (h->nx + 1) * (h->ny + 1);
    int32_t* order = h->vals[p.npass & 1];
    auto sort = [&](auto kernel, int nw, auto kin, const int32_t* vin) {
        const size_t lds = (sizeof(int) + nw * sizeof(uint16_t)) << p.shift;
        hipLaunchKernelGGL(kernel, dim3(p.buckets), dim3(nw * 64), lds, h->st, kin, vin, n, p.shift, ncell, h->total,
                           h->cstart, order);
    };
    // four waves hold a bucket of up to 5120 markers, eight one of 10240
    if (p.npass == 2) sort(k_cell_sort<8, uint32_t>, 8, (const uint32_t*)h->keys[0], h->vals[1]);
    else if (n / p.buckets <= 4096) sort(k_cell_sort<4, uint16_t>, 4, (const uint16_t*)h->keys[1], h->vals[0]);
    else sort(k_cell_sort<8, uint16_t>, 8, (const uint16_t*)h->keys[1], h->vals[0]);
    M_HIP(hipGetLastError());
    h->order = order;
    h->kind = kind;
    return TPH_OK;
}

tph_status tph_markers_to_grid(tph_markers* h, const double* phi_m, double fill, double* grid) {
    tph_internal_set_error_m("");
    if (!h || !grid || (h->n > 0 && !phi_m)) {
        tph_internal_set_error_m("handle, phi_m and grid are required");
        return TPH_ERR_INVALID;
    }
    if (h->kind < 0) {
        tph_internal_set_error_m("no binning: call tph_markers_bin first");
        return TPH_ERR_INVALID;
    }
    const NodeGrid q = node_grid(h, h->kind);
    if (h->n == 0) {
        const dim3 g((unsigned)((q.jmax - q.jmin + 1 + 255) / 256), (unsigned)(q.imax - q.imin + 1));
        hipLaunchKernelGGL(k_fill_nodes, g, dim3(256), 0, h->st, q, fill, grid);
        M_HIP(hipGetLastError());
        return TPH_OK;
    }
    const double ncell = (double)(h->nx + 1) * (h->ny + 1);
    const int R = ncell <= kRowCells ? 1 : 2, rows = kNodeWaves * R - 1;
    const dim3 g((unsigned)((h->nx + 1 + 62) / 63), (unsigned)((h->ny + 1 + rows - 1) / rows));
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, g, dim3(kNodeWaves * 64), 0, h->st, q, h->nx, h->ny, h->cstart, h->order, h->xm,
                           h->ym, phi_m, fill, grid);
    };
    // markers of 16 cells, with three deviations of a random placement; longer runs go in pieces of 320
    const double run = 16.0 * h->n / ncell, most = run + 3.0 * std::sqrt(run);
    if (R == 1) launch(most <= 128 ? k_nodes<1, 2> : most <= 192 ? k_nodes<1, 3> : most <= 256 ? k_nodes<1, 4> : k_nodes<1, 5>);
    else launch(most <= 128 ? k_nodes<2, 2> : most <= 192 ? k_nodes<2, 3> : most <= 256 ? k_nodes<2, 4> : k_nodes<2, 5>);
    M_HIP(hipGetLastError());
    return TPH_OK;
}

tph_status tph_markers_from_grid(tph_markers* h, int32_t kind, int32_t n, const double* xm, const double* ym,
                                 const double* grid, double* phi_m) {
    tph_internal_set_error_m("");
    if (!h || (n > 0 && (!xm || !ym || !grid || !phi_m))) {
        tph_internal_set_error_m("handle, xm, ym, grid and phi_m are required");
        return TPH_ERR_INVALID;
    }
    if (kind < TPH_NODES_BASIC || kind > TPH_NODES_VY || n < 0) {
        tph_internal_set_error_m("bad node kind or marker count");
        return TPH_ERR_INVALID;
    }
    if (n == 0) return TPH_OK;
    hipLaunchKernelGGL(k_from_grid, dim3(blocks(n)), dim3(256), 0, h->st, node_grid(h, kind), n, xm, ym, grid, phi_m);
    M_HIP(hipGetLastError());
    return TPH_OK;
}

tph_status tph_markers_advect_rk4(tph_markers* h, int32_t n, double* xm, double* ym, const double* vx,
                                  const double* vy, double dt) {
    tph_internal_set_error_m("");
    if (!h || (n > 0 && (!xm || !ym || !vx || !vy))) {
        tph_internal_set_error_m("handle, xm, ym, vx and vy are required");
        return TPH_ERR_INVALID;
    }
    if (n < 0 || !std::isfinite(dt)) {
        tph_internal_set_error_m("n must be >= 0 and dt finite");
        return TPH_ERR_INVALID;
    }
    if (n == 0) return TPH_OK;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(blocks(n)), dim3(256), 0, h->st, node_grid(h, TPH_NODES_VX),
                           node_grid(h, TPH_NODES_VY), h->lx, h->ly, n, xm, ym, vx, vy, dt);
    };
    if (n > kFewMarkers) launch(k_rk4<true>);
    else launch(k_rk4<false>);
    M_HIP(hipGetLastError());
    return TPH_OK;
}

tph_status tph_markers_sync(tph_markers* h) {
    tph_internal_set_error_m("");
    if (!h) {
        tph_internal_set_error_m("handle is NULL");
        return TPH_ERR_INVALID;
    }
    M_HIP(hipStreamSynchronize(h->st));
    return TPH_OK;
}

}  // extern "C"
