// Adjoint of the discrete Eikonal solve: dL/dF from dL/dT on the GPU.
//
// The paper solves the first-order Godunov system (Sec. 2.1, Eqs. 2-3) and
// does not differentiate it; this is an extension built on that
// discretisation.  At the forward solution every accepted non-seed point p
// with F_p > 0 satisfies, with u = |T| and U_p its upwind set (for each of the
// k axes whose values the local solver's root used, the neighbour on that
// axis with the smaller value),
//     sum_{q in U_p} w_q (u_p - u_q)^2 = (h / F_p)^2,
// (w_q = 1 / s^2 for a grid spacing h s along q's axis, 1 on a uniform grid)
// and its linearisation is
//     S_p du_p - sum_{q in U_p} w_q (u_p - u_q) du_q = -(h^2 / F_p^3) dF_p,
//     S_p = sum_{q in U_p} w_q (u_p - u_q).
// Seeds and points outside the accepted set are fixed.  The transposed system
// is solved exactly, in reverse dependency order: with lt_q = S_q lambda_q,
//     lt_q = dL/du_q + sum_{p : q in U_p} (w_q (u_p - u_q) / S_p) lt_p,
//     dL/dF_p = -(h^2 / (F_p^3 S_p)) lt_p,
// where dL/du = sign(T) dL/dT.  Since u_q < u_p for q in U_p, the dependency
// graph is acyclic: a point is final once all the points that used it are.
//
// GPU mapping.  A setup pass recomputes U_p from the final T (the same local
// solver as the forward march, so the same root and the same k) into 2 bits per
// axis.  All problems of a batch are then solved by one persistent cooperative
// kernel, in one of two forms:
// - the tile sweep (below): a wavefront takes an 8^3 tile into LDS and solves
//   every cell whose dependents are solved, until none is left; contributions
//   across a tile face go through HBM and list the neighbour tile for the next
//   phase;
// - the level sweep (planes and lines, whose tiles would be nearly empty, and
//   small workspaces): frontiers of points level by level; a point pushes its
//   contributions to its upwind points with FP64 atomics and decrements their
//   counters of unsolved dependents, and the point whose counter reaches zero
//   joins the next frontier.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "fmm_device.h"
#include "fmm_adjoint.h"

namespace fmm {

constexpr uint64_t ADJ_LOCAL_MASK = (1ull << 40) - 1;  // item = problem << 40 | local point

// The neighbours a point's root uses: a and pick hold per axis the smaller
// upwind value (+inf: none) and which neighbour it is (1 minus, 2 plus).
// Returns 2 bits per axis.  AN: some problem may have spacing factors.
template <bool AN = true>
__device__ __forceinline__ uint32_t upwind_pick(const Spacing &sp, const double a[3], const uint32_t pick[3], double r)
{
    int k = 0;
    if constexpr (AN)
        (void)local_solve(sp, a[0], a[1], a[2], r, &k);
    else
        (void)godunov_sel(a[0], a[1], a[2], r, &k);
    // the k smallest per-axis values, ties in axis order
    uint32_t code = 0;
#pragma unroll
    for (int ax = 0; ax < 3; ax++) {
        int rank = 0;
#pragma unroll
        for (int b = 0; b < 3; b++)
            if (b != ax && (a[b] < a[ax] || (a[b] == a[ax] && b < ax))) rank++;
        if (rank < k) code |= pick[ax] << (2 * ax);
    }
    return code;
}

// Upwind set of point p of problem I from the final values (the forward
// march's Alg. 11 filter and root): 2 bits per axis, 1 = the minus neighbour,
// 2 = the plus neighbour, 0 = not used.  Returns 0 when p is not an accepted
// non-seed point with F > 0 (or has no upwind value).
template <typename FT>
__device__ __forceinline__ uint32_t upwind_code(const AdjInst &I, int64_t p, int64_t i0, int64_t i1, int64_t i2)
{
    const uint8_t st = I.status[p];
    if ((st & 3u) != 2u) return 0;
    const double f = (double)((const FT *)I.F)[p];
    if (!(f > 0.0)) return 0;
    const double up = fabs(I.T[p]);
    const uint8_t side = st & 0x80u;
    const int64_t n[3] = {I.n0, I.n1, I.n2};
    const int64_t c[3] = {i0, i1, i2};
    const int64_t str[3] = {I.n1 * I.n2, I.n2, 1};
    double a[3];
    uint32_t pick[3];
#pragma unroll
    for (int ax = 0; ax < 3; ax++) {
        a[ax] = FMM_INF;
        pick[ax] = 0;
#pragma unroll
        for (int s = 0; s < 2; s++) {
            const bool in = s == 0 ? c[ax] > 0 : c[ax] + 1 < n[ax];
            if (!in) continue;
            const int64_t q = s == 0 ? p - str[ax] : p + str[ax];
            const uint8_t sq = I.status[q];
            if ((sq & 3u) < 2u || (sq & 0x80u) != side) continue;
            const double v = fabs(I.T[q]);
            if (v < up && v < a[ax]) {
                a[ax] = v;
                pick[ax] = (uint32_t)(s + 1);
            }
        }
    }
    return upwind_pick(I.sp, a, pick, I.h / f);
}

// dL/dF of a point with lt / S = lambda 2^e: -(h^2 / F^3) lambda 2^e, formed from
// mantissas and exponents apart.  h^2 / F^3 leaves the range of doubles for speeds
// beyond 1e+-102, though the gradient, about h lt / F^2, need not.  (An infinite
// speed's point is in the system where the march takes it as the largest finite
// one, next to a value of 0: its term is 0.)
__device__ __forceinline__ double adj_term(double h, double f, double lambda, int e)
{
    const double mf = __builtin_amdgcn_frexp_mant(f);
    const double q = quick_div(__builtin_amdgcn_frexp_mant(h), mf);  // h / F
    const int eq = __builtin_amdgcn_frexp_exp(h) - __builtin_amdgcn_frexp_exp(f);
    double m = quick_div(__builtin_amdgcn_frexp_mant(lambda) * q * q, mf);
    m = __builtin_amdgcn_class(lambda, 0x1 | 0x2 | 0x4 | 0x200) ? lambda : m;  // NaN and infinities
    m = f < FMM_INF ? m : 0.0 * lambda;
    return __builtin_amdgcn_ldexp(-m, __builtin_amdgcn_frexp_exp(lambda) + e + 2 * eq - __builtin_amdgcn_frexp_exp(f));
}

// Counter offset of points outside the linear system (see k_adj_setup).
constexpr uint32_t ADJ_FIXED_COUNT = 1u << 30;

// Reset: accumulators, counters and codes of every problem.
__global__ void k_adj_zero(AdjParams P, AdjInst I)
{
    const int64_t N = I.n0 * I.n1 * I.n2;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < N; p += (int64_t)gridDim.x * blockDim.x) {
        const int64_t g = I.base + p;
        P.acc[g] = 0.0;
        P.cnt[g] = 0u;
        P.code[g] = 0u;
    }
}

template <typename FT> __global__ void k_adj_setup(AdjParams P, AdjInst I)
{
    const int64_t N = I.n0 * I.n1 * I.n2;
    const int64_t n12 = I.n1 * I.n2;
    unsigned long long mine = 0;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < N; p += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i0 = p / n12, rem = p - i0 * n12, i1 = rem / I.n2, i2 = rem - i1 * I.n2;
        const uint32_t code = upwind_code<FT>(I, p, i0, i1, i2);
        if (!code) {
            // a fixed point (seed or outside the accepted set): its counter
            // starts far above the at most six decrements it can receive, so
            // it never reaches zero and never joins a frontier
            atomicAdd(&P.cnt[I.base + p], ADJ_FIXED_COUNT);
            continue;
        }
        mine++;
        const int64_t g = I.base + p;
        P.code[g] = (uint8_t)code;
        const double sgn = I.T[p] < 0.0 ? -1.0 : 1.0;
        P.acc[g] = sgn * I.dL_dT[p];
        const int64_t str[3] = {n12, I.n2, 1};
#pragma unroll
        for (int ax = 0; ax < 3; ax++) {
            const uint32_t c = (code >> (2 * ax)) & 3u;
            if (c) atomicAdd(&P.cnt[I.base + (c == 1 ? p - str[ax] : p + str[ax])], 1u);
        }
    }
    mine = wave_sum(mine);
    if ((threadIdx.x & 63) == 0 && mine) atomicAdd(&P.ctrl->n_points, mine);
}

// Wave-aggregated append of up to one item per lane.
__device__ __forceinline__ void push_item(bool want, uint64_t item, unsigned long long *len, uint64_t *list)
{
    const unsigned long long m = __ballot(want);
    if (!m) return;
    const int lane = threadIdx.x & 63;
    unsigned long long base = 0;
    const int leader = __ffsll((long long)m) - 1;
    if (lane == leader) base = atomicAdd(len, (unsigned long long)__popcll(m));
    base = __shfl(base, leader);
    if (want) list[base + (unsigned long long)__popcll(m & ((1ull << lane) - 1ull))] = item;
}

// First frontier: points in the system that no other point used.
__global__ void k_adj_front0(AdjParams P, AdjInst I, uint32_t j)
{
    const int64_t N = I.n0 * I.n1 * I.n2;
    const int64_t n_iter = (N + (int64_t)blockDim.x - 1) / blockDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n_iter;
         p += (int64_t)gridDim.x * blockDim.x) {
        bool want = false;
        if (p < N) {
            const int64_t g = I.base + p;
            want = P.code[g] != 0 && P.cnt[g] == 0;
        }
        push_item(want, ((uint64_t)j << 40) | (uint64_t)p, &P.ctrl->len[0], P.list0);
    }
}

#ifndef FMM_ADJ_WG_PER_CU
#define FMM_ADJ_WG_PER_CU 1
#endif
#ifndef FMM_ADJ_BLOCK
#define FMM_ADJ_BLOCK 256
#endif
constexpr int ADJ_BLOCK = FMM_ADJ_BLOCK;

// Process one frontier point: its gradient term, its contributions to its
// upwind points, and the upwind points whose last dependent it was join the
// next frontier (read only after the barrier that ends this level, so every
// contribution to them is complete).  New frontier entries are staged in LDS
// and appended with one atomic per workgroup.
template <typename FT>
__device__ __forceinline__ void adj_point(const AdjParams &P, uint64_t it, bool active, uint64_t *s_items,
                                          uint32_t *s_n)
{
    if (!active) return;
    const uint32_t j = (uint32_t)(it >> 40);
    const int64_t p = (int64_t)(it & ADJ_LOCAL_MASK);
    const AdjInst &I = P.inst[j];
    const int64_t g = I.base + p;
    const double lt = __hip_atomic_load(&P.acc[g], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t code = P.code[g];
    const double up = fabs(I.T[p]);
    const double f = (double)((const FT *)I.F)[p];
    const int64_t str[3] = {I.n1 * I.n2, I.n2, 1};
    int64_t q[3];
    double d[3];
    double S = 0.0;
#pragma unroll
    for (int ax = 0; ax < 3; ax++) {
        // weighted difference w_a (u_p - u_q), w_a = 1 / s_a^2 (1 on a uniform grid)
        const uint32_t cc = (code >> (2 * ax)) & 3u;
        const double w = I.sp.aniso ? 1.0 / (I.sp.s[ax] * I.sp.s[ax]) : 1.0;
        q[ax] = cc == 0 ? -1 : (cc == 1 ? p - str[ax] : p + str[ax]);
        d[ax] = cc == 0 ? 0.0 : w * (up - fabs(I.T[q[ax]]));
        S += d[ax];
    }
    // this point's gradient term; its accumulator is not needed any more
    P.acc[g] = adj_term(I.h, f, __builtin_amdgcn_frexp_mant(lt) / __builtin_amdgcn_frexp_mant(S),
                        __builtin_amdgcn_frexp_exp(lt) - __builtin_amdgcn_frexp_exp(S));
#pragma unroll
    for (int ax = 0; ax < 3; ax++) {
        if (q[ax] < 0) continue;
        const int64_t gq = I.base + q[ax];
        atomicAdd(&P.acc[gq], (d[ax] / S) * lt);
        // the last dependent of an upwind point in the system (fixed points
        // never count down to zero)
        const uint32_t old = atomicSub(&P.cnt[gq], 1u);
        if (old == 1u) s_items[atomicAdd(s_n, 1u)] = ((uint64_t)j << 40) | (uint64_t)q[ax];
    }
}

template <typename FT> __global__ void __launch_bounds__(ADJ_BLOCK) k_adj_sweep(AdjParams P)
{
    __shared__ uint32_t s_ok, s_n;
    __shared__ unsigned long long s_base;
    __shared__ uint64_t s_items[3 * ADJ_BLOCK];
    AdjCtrl *c = P.ctrl;
    const uint32_t nwg = gridDim.x;
    uint32_t gen = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) c->nwg = nwg;
    const uint64_t nth = (uint64_t)gridDim.x * blockDim.x;
    uint32_t level = 0;
    for (;;) {
        const unsigned long long n = ld_acq64(&c->len[level % 3]);
        if (n == 0) break;
        // the counter of the level after next is free: its last reader was
        // the previous level; the barrier below publishes the reset
        if (blockIdx.x == 0 && threadIdx.x == 0) c->len[(level + 2) % 3] = 0;
        const uint64_t *cur = (level & 1) ? P.list1 : P.list0;
        uint64_t *nxt = (level & 1) ? P.list0 : P.list1;
        unsigned long long *nlen = &c->len[(level + 1) % 3];
        // the pass count is uniform within a workgroup (barriers inside)
        for (unsigned long long k0 = (unsigned long long)blockIdx.x * blockDim.x; k0 < n; k0 += nth) {
            if (threadIdx.x == 0) s_n = 0;
            __syncthreads();
            const unsigned long long k = k0 + threadIdx.x;
            adj_point<FT>(P, k < n ? cur[k] : 0, k < n, s_items, &s_n);
            __syncthreads();
            const uint32_t m = s_n;
            if (threadIdx.x == 0 && m) s_base = atomicAdd(nlen, (unsigned long long)m);
            __syncthreads();
            for (uint32_t t = threadIdx.x; t < m; t += blockDim.x) nxt[s_base + t] = s_items[t];
            __syncthreads();
        }
        level++;
        if (!grid_sync(&c->bar, &c->abort, &c->error, ADJ_ERR_BARRIER, gen, nwg, &s_ok)) break;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) c->levels = level;
}

// dL/dF of one output array: the sum of the gradient terms of the problems
// that share it (a point outside a problem's system contributes 0).
__global__ void k_adj_gather(AdjParams P, AdjGather G)
{
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < G.n; p += (int64_t)gridDim.x * blockDim.x) {
        double s = G.accumulate ? G.out[p] : 0.0;
        for (uint32_t k = 0; k < G.m; k++) {
            const int64_t g = G.base[k] + p;
            if (P.code[g]) s += P.acc[g];
        }
        G.out[p] = s;
    }
}

__global__ void k_adj_init(AdjParams P, uint32_t n_inst)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        AdjCtrl *c = P.ctrl;
        c->bar = 0;
        c->abort = 0;
        c->error = 0;
        c->n_inst = n_inst;
        c->nwg = 0;
        c->levels = 0;
        c->len[0] = c->len[1] = c->len[2] = 0;
        c->n_points = 0;
        c->magic = ADJ_MAGIC;
    }
}

__global__ void k_adj_set_inst(AdjInst *dst, AdjPack<AdjInst> pk)
{
    const uint32_t k = threadIdx.x;
    if (k < pk.n) dst[pk.first + k] = pk.v[k];
}

// ---------------------------------------------------------------------------
// Host-side launcher.

static int adj_cus()
{
    static int cus = 0;
    if (!cus) {
        int dev = 0;
        (void)hipGetDevice(&dev);
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 1;
    }
    return cus;
}

// ---------------------------------------------------------------------------
// The tile sweep.
//
// Why tiles.  A level of the level sweep holds few points (256^3, 16 shots:
// 1.1e5 of 2.7e8 in each of 2481 levels), and costs a device barrier and six
// scattered atomics per point through memory.  A tile runs through many levels
// between two barriers, with its atomics in LDS: 400 phases instead of 2481
// levels, and only contributions across tile faces go through memory.  256^3,
// 16 shots: 150.4 ms with the level sweep, 43.1 ms with this one (setup 7.4 ms at
// 3.7 TB/s, sweep 34.7 ms, gather 0.95 ms at 4.6 TB/s).
//
// What bounds it.  A tile is activated 7.5 times (contributions arrive over
// several phases) and solves its cells in rounds of about 7, the width of its
// dependency graph: an activation is a serial chain of 12 rounds of about 1500
// cycles.  With the 10 tiles whose LDS fits a CU in flight the vector units are
// busy 40 % of the time and HBM moves 1.9 TB/s, so LDS space (tiles in flight)
// and the latency of a round are the limits, and the last phases, with few
// tiles, are bound by one activation's latency each (about 25 us).
//
// A wavefront holds one tile.  For counting, lane = row (x, y) of 8 cells along
// axis 2: which cells wait for a neighbour is a bit mask per row and direction,
// and the unsolved dependents of all cells are counted from them in registers.
// For solving, the ready cells are a queue in LDS and a lane takes one.
//
// Races.  A contribution is written once and read as one 8-byte word; a tile
// that reads a neighbour's face while that neighbour is writing it sees
// "waiting" or the final value, and the writer lists it for the next phase.
// The level travels in its own word, and a cell waits until both have
// arrived.

constexpr int ADJT_NW = 10;        // wavefronts per workgroup, one workgroup per CU (LDS)
constexpr uint32_t ADJT_SEGS = 8;  // work-list segments, one per XCD

struct AdjTileLds {
    double u[512 + 6 * 64];  // |T| of the cells, then the weighted differences across the faces
    double c[512];           // accumulated lt; solved cells: lambda = lt / S
    uint32_t lev[512];       // highest level among the dependents
    uint32_t cc[256];        // per cell 16 bits: unsolved dependents, then the upwind set (2 bits per axis)
    uint16_t queue[512];     // cells to solve: cell, then its upwind set
};

// Problem of tile t.
__device__ __forceinline__ uint32_t adj_tile_inst(const AdjTileParams &P, uint32_t t)
{
    uint32_t lo = 0, hi = P.n_inst;  // inst[lo].tbase <= t < inst[hi].tbase
    while (hi - lo > 1) {
        const uint32_t m = (lo + hi) / 2;
        if (P.inst[m].tbase <= t) lo = m;
        else hi = m;
    }
    return lo;
}

// Setup, one wavefront per tile: |T| and status of the tile and its face
// halo in LDS, the upwind set of every cell, and the tile's initial state.
// AN as in the sweep: without the weighted solver beside it the uniform one's
// registers do not spill (20 of them did; 256^3, 16 shots: 44.5 and 43.7 ms in all).
constexpr int ADJT_SETUP_WAVES = 4;
template <typename FT, bool AN>
__global__ void __launch_bounds__(ADJT_SETUP_WAVES * 64) __attribute__((amdgpu_waves_per_eu(4))) k_adjt_setup(AdjTileParams P)
{
    constexpr int D = 10, OX = 100, OY = 10, OZ = 1;
    __shared__ double s_u[ADJT_SETUP_WAVES][D * D * D];
    __shared__ uint8_t s_s[ADJT_SETUP_WAVES][D * D * D];
    const int lane = threadIdx.x & 63, wid = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double *U = s_u[wid];
    uint8_t *S = s_s[wid];
    const int a = lane >> 3, b = lane & 7;
    unsigned long long mine = 0;
    for (uint32_t t = blockIdx.x * ADJT_SETUP_WAVES + wid; t < P.ntiles; t += gridDim.x * ADJT_SETUP_WAVES) {
        const uint32_t j = __builtin_amdgcn_readfirstlane(P.n_inst == 1 ? 0u : adj_tile_inst(P, t));
        const AdjTileInst &I = P.inst[j];
        const uint32_t tl = t - I.tbase;
        const int64_t z0 = (int64_t)(tl % (uint32_t)I.t2) * 8;
        const int64_t y0 = (int64_t)((tl / (uint32_t)I.t2) % (uint32_t)I.t1) * 8;
        const int64_t x0 = (int64_t)(tl / ((uint32_t)I.t2 * (uint32_t)I.t1)) * 8;
        const FT *F = (const FT *)I.F;
        auto load = [&](int64_t i0, int64_t i1, int64_t i2, double &T, uint32_t &st) {
            T = 0.0;
            st = 0;  // outside the grid: never an upwind value
            if (i0 < 0 || i1 < 0 || i2 < 0 || i0 >= I.n0 || i1 >= I.n1 || i2 >= I.n2) return;
            const int64_t g = (i0 * I.n1 + i1) * I.n2 + i2;
            T = I.T[g];
            st = I.status[g];
        };
        // speed and loss gradient of a plane, requested one plane ahead
        FT fv = (FT)0;
        double gv = 0.0;
        const bool in12 = y0 + a < I.n1 && z0 + b < I.n2;
        auto load_plane = [&](int x) {
            if (!in12 || x0 + x >= I.n0) return;
            const int64_t p = ((x0 + x) * I.n1 + y0 + a) * I.n2 + z0 + b;
            fv = F[p];
            gv = I.dL_dT[p];
        };
        double tv[8], th[6];
        uint32_t sv[8], sh[6];
#pragma unroll
        for (int x = 0; x < 8; x++) load(x0 + x, y0 + a, z0 + b, tv[x], sv[x]);
        load_plane(0);
#pragma unroll
        for (int f = 0; f < 6; f++) {
            const int h = (f & 1) ? 8 : -1;
            load(x0 + (f < 2 ? h : a), y0 + (f < 2 ? a : f < 4 ? h : b), z0 + (f < 4 ? b : h), th[f], sh[f]);
        }
        wave_sync();  // the previous tile's reads are done
#pragma unroll
        for (int x = 0; x < 8; x++) {
            const int d = (x + 1) * OX + (a + 1) * OY + b + 1;
            U[d] = tv[x];
            S[d] = (uint8_t)sv[x];
        }
#pragma unroll
        for (int f = 0; f < 6; f++) {
            const int h = (f & 1) ? 9 : 0;
            const int d = (f < 2 ? h : a + 1) * OX + (f < 2 ? a + 1 : f < 4 ? h : b + 1) * OY + (f < 4 ? b + 1 : h);
            U[d] = th[f];
            S[d] = (uint8_t)sh[f];
        }
        wave_sync();
        const double w[3] = {AN && I.sp.aniso ? 1.0 / (I.sp.s[0] * I.sp.s[0]) : 1.0,
                             AN && I.sp.aniso ? 1.0 / (I.sp.s[1] * I.sp.s[1]) : 1.0,
                             AN && I.sp.aniso ? 1.0 / (I.sp.s[2] * I.sp.s[2]) : 1.0};
        uint64_t row = 0;
#pragma unroll 1
        for (int x = 0; x < 8; x++) {
            const int d = (x + 1) * OX + (a + 1) * OY + b + 1;
            const uint32_t st = S[d];
            const double tp = U[d], up = fabs(tp);
            const double f = (double)fv, gp = gv;
            if (x < 7) load_plane(x + 1);
            uint32_t code = 0;
            double g = 0.0;
            if ((st & 3u) == 2u) {
                if (f > 0.0) {
                    double v[3];
                    uint32_t pick[3];
#pragma unroll
                    for (int ax = 0; ax < 3; ax++) {
                        const int o = ax == 0 ? OX : ax == 1 ? OY : OZ;
                        const double lo = fabs(U[d - o]), hi = fabs(U[d + o]);
                        const uint32_t sl = S[d - o], sg = S[d + o];
                        v[ax] = FMM_INF;
                        pick[ax] = 0;
                        if ((sl & 3u) >= 2u && ((sl ^ st) & 0x80u) == 0 && lo < up) {
                            v[ax] = lo;
                            pick[ax] = 1;
                        }
                        if ((sg & 3u) >= 2u && ((sg ^ st) & 0x80u) == 0 && hi < up && hi < v[ax]) {
                            v[ax] = hi;
                            pick[ax] = 2;
                        }
                    }
                    code = upwind_pick<AN>(I.sp, v, pick, fast_div(I.h, f));
                    if (code) g = (tp < 0.0 ? -1.0 : 1.0) * gp;
                }
            }
            mine += code != 0;
            const size_t k = (size_t)t * 512 + x * 64 + lane;
            P.u[k] = up;
            P.c[k] = g;
            P.lev[k] = 0;
            // row words: byte r of a plane's ballot belongs to the row (x, r)
            uint64_t word = 0;
#pragma unroll
            for (int q = 0; q < 6; q++) {
                const unsigned long long m = __ballot((code >> q) & 1u);
                word |= ((m >> (8 * b)) & 0xFFull) << (8 * q);
            }
            word |= ((__ballot(code != 0) >> (8 * b)) & 0xFFull) << 56;
            if (a == x) row = word;
            // faces: the weighted difference to an upwind neighbour across it
#pragma unroll
            for (int f = 0; f < 6; f++) {
                const int ax = f >> 1;
                const int cc = ax == 0 ? x : ax == 1 ? a : b;
                if (cc != ((f & 1) ? 7 : 0)) continue;
                const int at = ax == 0 ? lane : ax == 1 ? x * 8 + b : x * 8 + a;
                const bool cross = ((code >> f) & 1u) != 0;
                const int o = ax == 0 ? OX : ax == 1 ? OY : OZ;
                const size_t q = ((size_t)t * 6 + f) * 64 + at;
                P.fw[q] = cross ? w[ax] * (up - fabs(U[(f & 1) ? d + o : d - o])) : 0.0;
                P.fo[q] = cross ? ADJT_WAIT : 0ull;
                P.fl[q] = cross ? ADJT_NOLEV : 0u;
            }
        }
        P.row[(size_t)t * 64 + lane] = row;
        if (lane == 0) {
            P.tag[t] = 0;
            uint32_t *h = P.head + (size_t)t * 16;
            h[0] = (uint32_t)I.t1 * (uint32_t)I.t2;
            h[1] = (uint32_t)I.t2;
            h[2] = (x0 > 0 ? 1u : 0u) | (x0 + 8 < I.n0 ? 2u : 0u) | (y0 > 0 ? 4u : 0u) | (y0 + 8 < I.n1 ? 8u : 0u) |
                   (z0 > 0 ? 16u : 0u) | (z0 + 8 < I.n2 ? 32u : 0u) | (I.sp.aniso ? 64u : 0u);
            h[3] = j;
        }
    }
    mine = wave_sum(mine);
    if (lane == 0 && mine) atomicAdd(&P.ctrl->n_points, mine);
}

struct AdjTileWave {
    uint32_t n, st;  // staged list appends: their number, and lane k's is entry k
    uint32_t level;  // highest level solved (per lane)
};

// Bits 0 to 3 of m as 0/1 in the four bytes of a word.
__device__ __forceinline__ uint32_t spread4(uint32_t m) { return ((m & 15u) * 0x00204081u) & 0x01010101u; }

// One activation of tile t: solve every cell whose dependents are solved.
// AN: some problem of the batch has per-axis spacing.
template <bool AN>
__device__ __forceinline__ void adj_tile(const AdjTileParams &P, AdjTileLds &L, uint32_t t, uint32_t phase,
                                         AdjTileWave &ws, unsigned long long *nlen, uint32_t *next)
{
    const int lane = threadIdx.x & 63, x = lane >> 3, y = lane & 7;
    // ---- loads.  The first phase visits every tile, most of which have no
    // ready cell yet: there the cells' values wait for that test.
    const bool visit = phase == 0;
    const uint32_t hv = lane < 16 ? P.head[(size_t)t * 16 + lane] : 0u;
    const uint64_t row = P.row[(size_t)t * 64 + lane];
    double uv[8], cv[8], wv[6];
    uint32_t lv[8];
    auto load_cells = [&]() {
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const size_t p = (size_t)t * 512 + k * 64 + lane;
            uv[k] = P.u[p];
            cv[k] = P.c[p];
            lv[k] = P.lev[p];
        }
#pragma unroll
        for (int f = 0; f < 6; f++) wv[f] = P.fw[((size_t)t * 6 + f) * 64 + lane];
    };
    auto stage_cells = [&]() {
#pragma unroll
        for (int k = 0; k < 8; k++) {
            L.u[k * 64 + lane] = uv[k];
            L.c[k * 64 + lane] = cv[k];
            L.lev[k * 64 + lane] = lv[k];
        }
#pragma unroll
        for (int f = 0; f < 6; f++) L.u[512 + f * 64 + lane] = wv[f];
    };
    if (!visit) load_cells();
    const uint32_t ts[3] = {(uint32_t)__builtin_amdgcn_readlane(hv, 0), (uint32_t)__builtin_amdgcn_readlane(hv, 1), 1u};
    const uint32_t flags = (uint32_t)__builtin_amdgcn_readlane(hv, 2);
    // contributions that may have arrived: the face cells that wait for one
    uint64_t fv[6];
    uint32_t fl[6];
#pragma unroll
    for (int f = 0; f < 6; f++) {
        uint64_t pend = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(hv, 4 + 2 * f) |
                        ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(hv, 5 + 2 * f) << 32);
        if (visit) pend = (flags >> f) & 1u ? ~0ull : 0ull;
        fv[f] = 0;
        fl[f] = 0;
        if (!((pend >> lane) & 1ull)) continue;
        const uint32_t nb = (f & 1) ? t + ts[f >> 1] : t - ts[f >> 1];
        const size_t q = ((size_t)nb * 6 + (f ^ 1)) * 64 + lane;
        fv[f] = __hip_atomic_load(&P.fo[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        fl[f] = __hip_atomic_load(&P.fl[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
    if (!visit) stage_cells();

    // ---- unsolved dependents of every cell of the row (4 + 4 byte counters).
    // A cell that is solved or outside the system starts at 64 and never
    // counts down to zero.
    const uint32_t lo = (uint32_t)row, hi = (uint32_t)(row >> 32);
    const uint32_t und = (hi >> 24) & ~(hi >> 16) & 0xFFu;  // unsolved cells of the row
    uint32_t n0 = spread4(~und) << 6, n1 = spread4(~und >> 4) << 6;
    auto count = [&](uint32_t m) {
        n0 += spread4(m);
        n1 += spread4(m >> 4);
    };
    {
        const uint32_t um = und * 0x01010101u;
        const uint32_t ulo = lo & um, uhi = hi & um;  // upwind masks of unsolved cells
        const uint32_t sxp = __shfl(ulo, x < 7 ? lane + 8 : lane), sxm = __shfl(ulo, x > 0 ? lane - 8 : lane);
        const uint32_t syp = __shfl(ulo, y < 7 ? lane + 1 : lane), sym = __shfl(ulo, y > 0 ? lane - 1 : lane);
        count(x < 7 ? sxp & 0xFFu : 0u);
        count(x > 0 ? (sxm >> 8) & 0xFFu : 0u);
        count(y < 7 ? (syp >> 16) & 0xFFu : 0u);
        count(y > 0 ? sym >> 24 : 0u);
        count((uhi & 0xFFu) >> 1);
        count(((uhi >> 8) << 1) & 0xFFu);
    }
    uint64_t left = 0;   // lane f: the cells of face f that go on waiting
    uint32_t take = 0;   // bit f: this lane's contribution across face f has arrived
#pragma unroll
    for (int f = 0; f < 6; f++) {
        const bool wait = fv[f] == ADJT_WAIT || fl[f] == ADJT_NOLEV;
        const uint64_t still = __ballot(wait);
        if (fl[f] != 0 && !wait) take |= 1u << f;
        if (lane == f) left = still;
        uint32_t m;
        if (f < 2)
            m = x == (f == 0 ? 0 : 7) ? (uint32_t)(still >> (8 * y)) & 0xFFu : 0u;
        else if (f < 4)
            m = y == (f == 2 ? 0 : 7) ? (uint32_t)(still >> (8 * x)) & 0xFFu : 0u;
        else
            m = (wait ? 1u : 0u) << (f == 4 ? 0 : 7);
        count(m);
    }
    // ready: the bytes that are zero (counters are below 128)
    const uint32_t z0 = ((n0 + 0x7F7F7F7Fu) & 0x80808080u) ^ 0x80808080u;
    const uint32_t z1 = ((n1 + 0x7F7F7F7Fu) & 0x80808080u) ^ 0x80808080u;
    const bool any = __ballot((z0 | z1) != 0) != 0;
    if (!any) {
        // contributions that have arrived are left for a later visit
        if (visit) {
            uint64_t w = 0;
#pragma unroll
            for (int f = 0; f < 6; f++) {
                const uint64_t m = __ballot(fl[f] != 0);
                if (lane == f) w = m;
            }
            if (lane < 6) *(uint64_t *)&P.head[(size_t)t * 16 + 4 + 2 * lane] = w;
        }
        return;
    }
    if (lane < 6) *(uint64_t *)&P.head[(size_t)t * 16 + 4 + 2 * lane] = left;
    if (visit) {
        load_cells();
        stage_cells();
    }

    // ---- counters, upwind sets and the ready cells
    uint32_t code0 = 0, code1 = 0;
#pragma unroll
    for (int k = 0; k < 6; k++) {
        const uint32_t m = k < 4 ? lo >> (8 * k) : hi >> (8 * (k - 4));
        code0 |= spread4(m) << k;
        code1 |= spread4(m >> 4) << k;
    }
    L.cc[lane * 4 + 0] = __builtin_amdgcn_perm(code0, n0, 0x05010400u);
    L.cc[lane * 4 + 1] = __builtin_amdgcn_perm(code0, n0, 0x07030602u);
    L.cc[lane * 4 + 2] = __builtin_amdgcn_perm(code1, n1, 0x05010400u);
    L.cc[lane * 4 + 3] = __builtin_amdgcn_perm(code1, n1, 0x07030602u);
    uint32_t tail = 0;  // queue entries (wave-uniform)
    auto push = [&](bool want, uint32_t entry) {
        const unsigned long long m = __ballot(want);
        if (want)
            L.queue[tail + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                (uint16_t)entry;
        tail += (uint32_t)__popcll(m);
    };
#pragma unroll
    for (int k = 0; k < 8; k++)
        push((((k < 4 ? z0 : z1) >> (8 * (k & 3) + 7)) & 1u) != 0,
             (uint32_t)(lane * 8 + k) | ((((k < 4 ? code0 : code1) >> (8 * (k & 3))) & 63u) << 9));
    wave_sync();
    // contributions that have arrived across the faces (x, then y, then z)
#pragma unroll
    for (int f = 0; f < 6; f++) {
        if ((take >> f) & 1u) {
            const int q = f < 2 ? (f == 0 ? 0 : 448) + lane : f < 4 ? x * 64 + (f == 2 ? 0 : 56) + y : lane * 8 + (f == 4 ? 0 : 7);
            L.c[q] += bitsd(fv[f]);
            L.lev[q] = max(L.lev[q], fl[f]);
        }
        wave_sync();  // a cell on two faces
    }

    // ---- solve.  A queued cell is final: it passes its weighted lambda on to
    // its upwind cells, and the one whose last dependent it was joins the queue.
    double w[3] = {1.0, 1.0, 1.0};
    if (AN && (flags & 64u)) {
        const AdjInst &I = P.inst[__builtin_amdgcn_readlane(hv, 3)];
#pragma unroll
        for (int ax = 0; ax < 3; ax++) w[ax] = 1.0 / (I.sp.s[ax] * I.sp.s[ax]);
    }
    uint32_t sent = 0, head = 0;
    while (head < tail) {
        const uint32_t i = head + (uint32_t)lane;
        const bool act = i < tail;
        head = min(head + 64u, tail);
        bool last[3] = {false, false, false};
        uint32_t entry[3] = {0, 0, 0};
        if (act) {
            const uint32_t e = L.queue[i];
            const int q = (int)(e & 511u);
            const uint32_t code = e >> 9;
            const int qx = q >> 6, qy = (q >> 3) & 7, qz = q & 7;
            int tgt[3];
            bool in[3];
            uint32_t cross = 0;
            double v[3], d[3];
            // all reads in one LDS round trip; an axis that is not used reads
            // the cell itself (difference 0)
            const double uq = L.u[q], lt = L.c[q];
            const uint32_t lev = L.lev[q] + 1u;
#pragma unroll
            for (int ax = 0; ax < 3; ax++) {
                const uint32_t c2 = (code >> (2 * ax)) & 3u;
                const int co = ax == 0 ? qx : ax == 1 ? qy : qz, off = ax == 0 ? 64 : ax == 1 ? 8 : 1;
                const int at = ax == 0 ? q & 63 : ax == 1 ? qx * 8 + qz : q >> 3;
                const bool plus = c2 == 2u, edge = co == (plus ? 7 : 0);
                in[ax] = c2 != 0 && !edge;
                if (c2 != 0 && edge) cross |= c2 << (2 * ax);
                tgt[ax] = plus ? q + off : q - off;
                const int ext = 512 + (2 * ax) * 64 + at + (plus ? 64 : 0);
                v[ax] = L.u[c2 == 0 ? q : edge ? ext : tgt[ax]];
            }
            ws.level = max(ws.level, lev);
#pragma unroll
            for (int ax = 0; ax < 3; ax++) {
                const double dif = AN ? w[ax] * (uq - v[ax]) : uq - v[ax];
                d[ax] = (cross >> (2 * ax)) & 3u ? v[ax] : dif;
            }
            // lambda = lt / S, and d lambda to each upwind cell.  Where lambda
            // leaves the range of normal numbers (lt = 0 apart) the weights d / S
            // are formed first, and lambda is kept as mantissa and exponent.
            const double S = (d[0] + d[1]) + d[2];
            double c = quick_div(lt, S);
            double p[3] = {d[0] * c, d[1] * c, d[2] * c};
            // signalling and quiet NaN; those, infinities, subnormals and zeros
            const bool nan = __builtin_amdgcn_class(c, 0x1 | 0x2);
            const bool odd = __builtin_amdgcn_class(c, 0x1 | 0x2 | 0x4 | 0x10 | 0x20 | 0x40 | 0x80 | 0x200);
            // (below 2^-960 the quotient's remainder may underflow)
            const int rare = (int)nan | (((int)odd | (int)(fabs(lt) < 0x1p-960)) & (int)(lt != 0.0));
            if (__builtin_expect(rare, 0)) {
                asm volatile("");
#pragma unroll
                for (int ax = 0; ax < 3; ax++) p[ax] = (d[ax] / S) * lt;
                c = __builtin_amdgcn_frexp_mant(lt) / __builtin_amdgcn_frexp_mant(S);
                const int e = __builtin_amdgcn_frexp_exp(lt) - __builtin_amdgcn_frexp_exp(S);
                L.lev[q] = ADJT_SCALED | (uint32_t)(e + ADJT_BIAS);  // no longer read as a level
                sent |= 64u;
            }
            L.c[q] = c;
#pragma unroll
            for (int ax = 0; ax < 3; ax++) {
                if (!in[ax]) continue;
                __hip_atomic_fetch_add(&L.c[tgt[ax]], p[ax], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                __hip_atomic_fetch_max(&L.lev[tgt[ax]], lev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            }
            // the contributions come before the counters (LDS works in order)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            uint32_t old[3];
#pragma unroll
            for (int ax = 0; ax < 3; ax++) {
                // an axis that is not passed on counts the cell's own word down by nothing
                const int to = in[ax] ? tgt[ax] : q;
                old[ax] = __hip_atomic_fetch_sub(&L.cc[to >> 1], in[ax] ? 1u << (16 * (to & 1)) : 0u, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WAVEFRONT);
            }
            if (cross) {
#pragma unroll
                for (int ax = 0; ax < 3; ax++) {
                    const uint32_t c2 = (cross >> (2 * ax)) & 3u;
                    if (!c2) continue;
                    const uint32_t f = 2 * ax + (c2 >> 1);
                    const int at = ax == 0 ? q & 63 : ax == 1 ? qx * 8 + qz : q >> 3;
                    uint64_t b = bits_of(p[ax]);
                    if (b == ADJT_WAIT) b = 0x7ff8000000000000ull;  // a NaN whose bits mean "waiting"
                    const size_t o = ((size_t)t * 6 + f) * 64 + at;
                    __hip_atomic_store(&P.fo[o], b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                    __hip_atomic_store(&P.fl[o], lev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                    sent |= 1u << f;
                }
            }
#pragma unroll
            for (int ax = 0; ax < 3; ax++) {
                const uint32_t o16 = old[ax] >> (16 * (tgt[ax] & 1));
                last[ax] = in[ax] && (o16 & 0xFFu) == 1u;
                entry[ax] = (uint32_t)tgt[ax] | (((o16 >> 8) & 63u) << 9);
            }
        }
#pragma unroll
        for (int ax = 0; ax < 3; ax++) push(last[ax], entry[ax]);
        wave_sync();
    }

    // ---- list the tiles that got contributions; write back (a cell is solved
    // when its counter is zero).  The listing waits for its reply before the
    // write-back's stores are issued, so that it does not wait for them.
    uint32_t nb = 0;
    bool want = false;
#pragma unroll
    for (int f = 0; f < 6; f++) {
        const bool any_f = __ballot((sent >> f) & 1u) != 0;
        if (lane == f && any_f) {
            nb = (f & 1) ? t + ts[f >> 1] : t - ts[f >> 1];
            want = true;
        }
    }
    if (__ballot((sent >> 6) & 1u) != 0 && lane == 0) P.head[(size_t)t * 16 + 2] = flags | 128u;
    if (want) want = atomicExch(&P.tag[nb], phase + 1u) != phase + 1u;
    const unsigned long long m = __ballot(want);
    const uint32_t cnt = (uint32_t)__popcll(m);
    if (ws.n + cnt > 64u) {
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(nlen, (unsigned long long)ws.n);
        base = bcast0(base);
        if (lane < (int)ws.n) next[base + lane] = ws.st;
        ws.n = 0;
    }
#pragma unroll
    for (int f = 0; f < 6; f++) {
        if (!((m >> f) & 1ull)) continue;
        const uint32_t v = (uint32_t)__builtin_amdgcn_readlane(nb, f);
        if (lane == (int)ws.n) ws.st = v;
        ws.n++;
    }
    uint32_t solved = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const uint32_t e = L.cc[lane * 4 + k];
        solved |= ((e & 0xFFu) == 0 ? 1u : 0u) << (2 * k);
        solved |= ((e & 0xFF0000u) == 0 ? 1u : 0u) << (2 * k + 1);
    }
    P.row[(size_t)t * 64 + lane] = row | ((uint64_t)solved << 48);
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const int q = k * 64 + lane;
        const uint32_t cn = ((const uint16_t *)L.cc)[q] & 0xFFu;
        const double v = L.c[q];
        const uint32_t l = L.lev[q];
        if (cn < 58u) {  // not solved before this activation
            P.c[(size_t)t * 512 + q] = v;
            P.lev[(size_t)t * 512 + q] = l;
        }
    }
    wave_sync();
}

template <bool AN>
__global__ void __launch_bounds__(ADJT_NW * 64) __attribute__((amdgpu_waves_per_eu(3))) k_adjt_sweep(AdjTileParams P)
{
    __shared__ AdjTileLds s_tile[ADJT_NW];
    __shared__ uint32_t s_ok, s_drained, s_cnt[ADJT_NW];
    __shared__ unsigned long long s_base;
    AdjTileCtrl *c = P.ctrl;
    const int lane = threadIdx.x & 63, wid = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    AdjTileLds &L = s_tile[wid];
    const uint32_t nwg = gridDim.x, nseg = nwg < ADJT_SEGS ? nwg : ADJT_SEGS;
    uint32_t gen = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) c->nwg = nwg;
    if (threadIdx.x == 0) s_drained = 0;
    __syncthreads();
    AdjTileWave ws;
    ws.n = ws.st = 0;
    ws.level = 0;
    // Phase 0 visits every tile, a later phase the tiles that were listed.
    // Phases are numbered with 32 bits; a solve has at most as many as points
    // on its longest dependency chain.
    uint32_t phase = 0;
    uint64_t n = P.ntiles;
    for (;;) {
        // counters of the next phase, last read two barriers ago
        if (blockIdx.x == 0) {
            if (threadIdx.x == 0) c->len[(phase + 2) % 3] = 0;
            if (threadIdx.x < ADJT_SEGS) c->work[(phase + 1) % 3][threadIdx.x][0] = 0;
        }
        const uint32_t *items = (phase & 1u) ? P.list1 : P.list0;
        uint32_t *next = (phase & 1u) ? P.list0 : P.list1;
        unsigned long long *nlen = &c->len[(phase + 1) % 3];
        // work distribution as in the forward driver: the first items of a
        // segment belong to its wavefronts, the rest are claimed
        uint32_t(*work)[32] = c->work[phase % 3];
        auto seg_lo = [&](uint32_t s) { return (uint32_t)((n * s) / nseg); };
        auto seg_own = [&](uint32_t s) { return (nwg - s + nseg - 1) / nseg * (uint32_t)ADJT_NW; };
        uint32_t seg = blockIdx.x % nseg, left = nseg, claim = 0;
        uint32_t lo = seg_lo(seg), len = seg_lo(seg + 1) - lo, own = seg_own(seg);
        uint32_t k = (uint32_t)wid * (own / ADJT_NW) + blockIdx.x / nseg;
        for (bool first = true;; first = false) {
            if (!first) k = len > own ? own + bcast0(claim) : len;
            if (k >= len) {
                if (len > own && lane == 0) atomicOr(&s_drained, 1u << seg);
                const uint32_t gone = __builtin_amdgcn_readfirstlane(*(volatile uint32_t *)&s_drained);
                bool found = false;
                while (!found && --left > 0) {
                    seg = seg + 1 == nseg ? 0 : seg + 1;
                    lo = seg_lo(seg);
                    len = seg_lo(seg + 1) - lo;
                    own = seg_own(seg);
                    found = len > own && !((gone >> seg) & 1u);
                }
                if (!found) break;
                if (lane == 0) claim = atomicAdd(&work[seg][0], 1u);
                continue;
            }
            if (len > own && lane == 0) claim = atomicAdd(&work[seg][0], 1u);
            const uint32_t t = phase ? __builtin_amdgcn_readfirstlane(items[lo + k]) : lo + k;
            adj_tile<AN>(P, L, __builtin_amdgcn_readfirstlane(t), phase, ws, nlen, next);
        }
        // one append per workgroup for what its wavefronts still hold
        if (lane == 0) s_cnt[wid] = ws.n;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t tot = 0;
            for (int q = 0; q < ADJT_NW; q++) tot += s_cnt[q];
            s_base = tot ? atomicAdd(nlen, (unsigned long long)tot) : 0ull;
            s_drained = 0;
        }
        __syncthreads();
        unsigned long long at = s_base;
        for (int q = 0; q < wid; q++) at += s_cnt[q];
        if (lane < (int)ws.n) next[at + lane] = ws.st;
        ws.n = 0;
        if (!grid_sync(&c->bar, &c->abort, &c->error, ADJ_ERR_BARRIER, gen, nwg, &s_ok)) break;
        phase++;
        n = ld_acq64(&c->len[phase % 3]);
        if (n == 0) break;
    }
    uint32_t lev = ws.level;
    for (int o = 32; o > 0; o >>= 1) lev = max(lev, (uint32_t)__shfl_xor(lev, o));
    if (lane == 0 && lev) atomicMax(&c->levels, lev);
}

// dL/dF of one output array, one wavefront per tile: the sum of the gradient
// terms of the problems that share it.  Bound by memory; with six wavefronts per
// SIMD 0.95 ms at 256^3 with 16 shots (4.6 TB/s), with five 1.11.
template <typename FT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6)))
k_adjt_gather(AdjTileParams P, AdjTileGather G)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int a = lane >> 3, b = lane & 7;
    const uint32_t nt = (uint32_t)G.t0 * (uint32_t)G.t1 * (uint32_t)G.t2;
    for (uint32_t t = blockIdx.x * 4 + wid; t < nt; t += gridDim.x * 4) {
        const int64_t z0 = (int64_t)(t % (uint32_t)G.t2) * 8;
        const int64_t y0 = (int64_t)((t / (uint32_t)G.t2) % (uint32_t)G.t1) * 8;
        const int64_t x0 = (int64_t)(t / ((uint32_t)G.t2 * (uint32_t)G.t1)) * 8;
        const bool in12 = y0 + a < G.n1 && z0 + b < G.n2;
        double s[8];
#pragma unroll
        for (int x = 0; x < 8; x++) {
            s[x] = 0.0;
            if (G.accumulate && in12 && x0 + x < G.n0) s[x] = G.out[((x0 + x) * G.n1 + y0 + a) * G.n2 + z0 + b];
        }
        for (uint32_t k = 0; k < G.m; k++) {
            const size_t tk = (size_t)G.tbase[k] + t;
            const FT *F = (const FT *)G.F[k];
            const bool scaled = (P.head[tk * 16 + 2] & 128u) != 0;
#pragma unroll
            for (int x = 0; x < 8; x++) {
                // the row word's system byte; inside the system the point is in the grid
                const uint32_t sys = (uint32_t)(P.row[tk * 64 + x * 8 + a] >> 56);
                if (!((sys >> b) & 1u)) continue;
                const double f = (double)F[((x0 + x) * G.n1 + y0 + a) * G.n2 + z0 + b];
                int e = 0;
                if (scaled) {
                    const uint32_t l = P.lev[tk * 512 + x * 64 + lane];
                    if (l & ADJT_SCALED) e = (int)(l & ~ADJT_SCALED) - ADJT_BIAS;
                }
                s[x] += adj_term(G.h[k], f, P.c[tk * 512 + x * 64 + lane], e);
            }
        }
#pragma unroll
        for (int x = 0; x < 8; x++)
            if (in12 && x0 + x < G.n0) G.out[((x0 + x) * G.n1 + y0 + a) * G.n2 + z0 + b] = s[x];
    }
}

// The control block; with the first problem descriptors.
__global__ void k_adjt_init(AdjTileParams P, AdjPack<AdjTileInst> pk)
{
    const uint32_t k = threadIdx.x;
    if (pk.first == 0) {
        AdjTileCtrl *c = P.ctrl;
        if (k == 0) {
            c->bar = 0;
            c->abort = 0;
            c->error = 0;
            c->n_inst = P.n_inst;
            c->nwg = 0;
            c->levels = 0;
            c->len[0] = c->len[1] = c->len[2] = 0;
            c->n_points = 0;
            c->magic = ADJ_MAGIC;
        }
        if (k < 3 * ADJT_SEGS) c->work[k / ADJT_SEGS][k % ADJT_SEGS][0] = 0;
    }
    if (k < pk.n) ((AdjTileInst *)P.inst)[pk.first + k] = pk.v[k];
}

template <typename FT> static hipError_t launch_adjoint_t(const AdjParams &P, const AdjTileInst *insts, int64_t n,
                                                       hipStream_t s)
{
    const int cus = adj_cus();
    hipError_t e;
    hipLaunchKernelGGL(k_adj_init, dim3(1), dim3(64), 0, s, P, (uint32_t)n);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int64_t first = 0; first < n; first += ADJ_PACK) {
        AdjPack<AdjInst> pk;
        memset(&pk, 0, sizeof pk);
        pk.first = (uint32_t)first;
        pk.n = (uint32_t)std::min<int64_t>(ADJ_PACK, n - first);
        for (uint32_t k = 0; k < pk.n; k++) pk.v[k] = insts[first + k];
        hipLaunchKernelGGL(k_adj_set_inst, dim3(1), dim3(64), 0, s, (AdjInst *)P.inst, pk);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    auto blocks_for = [&](const AdjInst &I) {
        const int64_t N = I.n0 * I.n1 * I.n2;
        return (unsigned)std::max<int64_t>(1, std::min<int64_t>((N + 255) / 256, (int64_t)cus * 16));
    };
    for (int64_t j = 0; j < n; j++) {
        hipLaunchKernelGGL(k_adj_zero, dim3(blocks_for(insts[j])), dim3(256), 0, s, P, insts[j]);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    for (int64_t j = 0; j < n; j++) {
        hipLaunchKernelGGL(k_adj_setup<FT>, dim3(blocks_for(insts[j])), dim3(256), 0, s, P, insts[j]);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    for (int64_t j = 0; j < n; j++) {
        hipLaunchKernelGGL(k_adj_front0, dim3(blocks_for(insts[j])), dim3(256), 0, s, P, insts[j], (uint32_t)j);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    static int occ = -1;
    auto kern = k_adj_sweep<FT>;
    if (occ < 0) {
        int nb = 0;
        if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, ADJ_BLOCK, 0)) != hipSuccess) return e;
        occ = nb;
    }
    if (occ <= 0) return hipErrorInvalidConfiguration;
    const unsigned grid = (unsigned)(std::min(occ, FMM_ADJ_WG_PER_CU) * cus);
    AdjParams Pc = P;
    void *args[] = {&Pc};
    if ((e = launch_coresident((const void *)kern, dim3(grid), dim3(ADJ_BLOCK), args, s)) != hipSuccess) return e;
    // gather each output array over the problems that share it
    std::vector<bool> done((size_t)n, false);
    for (int64_t j = 0; j < n; j++) {
        if (done[(size_t)j]) continue;
        AdjGather G;
        memset(&G, 0, sizeof G);
        G.out = insts[j].dL_dF;
        G.n = insts[j].n0 * insts[j].n1 * insts[j].n2;
        for (int64_t k = j; k < n; k++) {
            if (done[(size_t)k] || insts[k].dL_dF != G.out) continue;
            done[(size_t)k] = true;
            G.base[G.m++] = insts[k].base;
            if (G.m == ADJ_GATHER) {
                hipLaunchKernelGGL(k_adj_gather, dim3(blocks_for(insts[j])), dim3(256), 0, s, P, G);
                if ((e = hipGetLastError()) != hipSuccess) return e;
                G.accumulate = 1;
                G.m = 0;
            }
        }
        if (G.m) {
            hipLaunchKernelGGL(k_adj_gather, dim3(blocks_for(insts[j])), dim3(256), 0, s, P, G);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

hipError_t launch_adjoint(const AdjParams &P, const AdjTileInst *insts, int64_t n, bool f64, hipStream_t s)
{
    return f64 ? launch_adjoint_t<double>(P, insts, n, s) : launch_adjoint_t<float>(P, insts, n, s);
}

template <bool AN> static hipError_t launch_sweep(const AdjTileParams &P, hipStream_t s)
{
    static int occ = -1;
    auto kern = k_adjt_sweep<AN>;
    if (occ < 0) {
        int nb = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, ADJT_NW * 64, 0);
        if (e != hipSuccess) return e;
        occ = nb;
    }
    if (occ <= 0) return hipErrorInvalidConfiguration;
    AdjTileParams Pc = P;
    void *args[] = {&Pc};
    // a workgroup per CU, fewer if there are not eight tiles for each (as in
    // the forward driver: the barrier is cheaper)
    const unsigned grid = std::min((unsigned)adj_cus(), (P.ntiles + 7u) / 8u);
    return launch_coresident((const void *)kern, dim3(grid), dim3(ADJT_NW * 64), args, s);
}

template <typename FT> static hipError_t launch_adjoint_tiles_t(const AdjTileParams &P, const AdjTileInst *insts, int64_t n,
                                                               hipStream_t s)
{
    const int cus = adj_cus();
    hipError_t e;
    for (int64_t first = 0; first < n; first += ADJ_PACK) {
        AdjPack<AdjTileInst> pk;
        memset(&pk, 0, sizeof pk);
        pk.first = (uint32_t)first;
        pk.n = (uint32_t)std::min<int64_t>(ADJ_PACK, n - first);
        for (uint32_t k = 0; k < pk.n; k++) pk.v[k] = insts[first + k];
        hipLaunchKernelGGL(k_adjt_init, dim3(1), dim3(64), 0, s, P, pk);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const unsigned sb = (unsigned)std::min<int64_t>(((int64_t)P.ntiles + ADJT_SETUP_WAVES - 1) / ADJT_SETUP_WAVES,
                                                    (int64_t)cus * 16);
    bool aniso = false;
    for (int64_t j = 0; j < n; j++) aniso |= insts[j].sp.aniso != 0;
    if (aniso)
        hipLaunchKernelGGL((k_adjt_setup<FT, true>), dim3(sb), dim3(ADJT_SETUP_WAVES * 64), 0, s, P);
    else
        hipLaunchKernelGGL((k_adjt_setup<FT, false>), dim3(sb), dim3(ADJT_SETUP_WAVES * 64), 0, s, P);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = aniso ? launch_sweep<true>(P, s) : launch_sweep<false>(P, s)) != hipSuccess) return e;
    // gather each output array over the problems that share it
    std::vector<bool> done((size_t)n, false);
    for (int64_t j = 0; j < n; j++) {
        if (done[(size_t)j]) continue;
        const AdjTileInst &J = insts[j];
        AdjTileGather G;
        memset(&G, 0, sizeof G);
        G.out = J.dL_dF;
        G.n0 = J.n0;
        G.n1 = J.n1;
        G.n2 = J.n2;
        G.t0 = J.t0;
        G.t1 = J.t1;
        G.t2 = J.t2;
        const int64_t nt = (int64_t)J.t0 * J.t1 * J.t2;
        const unsigned gb = (unsigned)std::min<int64_t>((nt + 3) / 4, (int64_t)cus * 16);
        for (int64_t k = j; k < n; k++) {
            if (!done[(size_t)k] && insts[k].dL_dF == G.out) {
                done[(size_t)k] = true;
                G.tbase[G.m] = insts[k].tbase;
                G.F[G.m] = insts[k].F;
                G.h[G.m] = insts[k].h;
                G.m++;
            }
            if (G.m == ADJ_GATHER || (k == n - 1 && G.m)) {
                hipLaunchKernelGGL(k_adjt_gather<FT>, dim3(gb), dim3(256), 0, s, P, G);
                if ((e = hipGetLastError()) != hipSuccess) return e;
                G.accumulate = 1;
                G.m = 0;
            }
        }
    }
    return hipSuccess;
}

hipError_t launch_adjoint_tiles(const AdjTileParams &P, const AdjTileInst *insts, int64_t n, bool f64, hipStream_t s)
{
    return f64 ? launch_adjoint_tiles_t<double>(P, insts, n, s) : launch_adjoint_tiles_t<float>(P, insts, n, s);
}

}  // namespace fmm
