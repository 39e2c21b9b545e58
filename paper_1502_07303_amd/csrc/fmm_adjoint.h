// Internal definitions of the adjoint kernels (fmm_adjoint.hip) shared with
// the host side of libfmm.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "fmm_device.h"

namespace fmm {

// One problem of an adjoint batch (device copy).  Arrays are the caller's,
// row-major (n0, n1, n2).
struct AdjInst {
    int64_t n0, n1, n2;
    int64_t base;  // global index of the problem's first point in the level sweep's arrays
    double h;
    const void *F;
    const double *T;
    const uint8_t *status;
    const double *dL_dT;
    double *dL_dF;
    Spacing sp;  // per-axis spacing factors (weights 1 / s^2)
};

// The same for the tile sweep.
struct AdjTileInst : AdjInst {
    int32_t t0, t1, t2;  // 8^3 tiles per axis
    uint32_t tbase;      // global index of the problem's first tile
};

enum : uint32_t { ADJ_ERR_BARRIER = 32u };
constexpr uint32_t ADJ_MAGIC = 0x41444a31u;

struct AdjCtrl {
    alignas(128) uint32_t bar;  // grid barrier arrivals (monotonic)
    alignas(128) uint32_t abort;
    uint32_t error;
    uint32_t n_inst;
    uint32_t nwg;
    uint32_t levels;                  // frontier levels processed
    uint32_t magic;                   // ADJ_MAGIC once a run has initialised the workspace
    alignas(128) unsigned long long len[3];  // frontier lengths, by level mod 3
    alignas(128) unsigned long long n_points;  // points of the linear system
};

// The tile sweep's adds claim counters of the phases (by phase mod 3), one per
// segment of the work list and 128 B apart.
struct AdjTileCtrl : AdjCtrl {
    alignas(128) uint32_t work[3][8][32];
};

// Callers size workspaces by the level sweep's structures.
static_assert(sizeof(AdjCtrl) == 512 && sizeof(AdjInst) == 112, "part of the workspace layout");

struct AdjParams {
    AdjCtrl *ctrl;
    const AdjInst *inst;
    double *acc;      // per point: S_p lambda_p being accumulated; once processed, its dL/dF term
    uint32_t *cnt;    // per point: dependents not yet processed
    uint8_t *code;    // per point: upwind set, 2 bits per axis
    uint64_t *list0, *list1;  // frontiers
};

// The tile sweep's state: per 8^3 tile, 64 rows (x, y) of 8 cells along axis 2.
// A row word holds, one bit per cell: bytes 0 to 5 the cells whose upwind
// neighbour on axis 0, 1, 2 is the minus (even bytes) or plus (odd bytes) one,
// byte 6 the cells that are solved and byte 7 the cells of the linear system.
struct AdjTileParams {
    AdjTileCtrl *ctrl;
    const AdjTileInst *inst;
    uint32_t n_inst, ntiles;
    // 16 words per tile: tile strides along axes 0 and 1, flags (bits 0 to 5:
    // there is a tile across face f; bit 6: per-axis spacing; bit 7: some lambda
    // is scaled), problem, and per face 64 bits for the cells that wait for a contribution across it
    uint32_t *head;
    uint64_t *row;    // 64 row words per tile
    double *u;        // |T|
    double *c;        // sign(T) dL/dT until the cell is solved, then lambda = lt / S
    uint32_t *lev;    // dependency level of a solved cell (1: no dependents), or
                      // ADJT_SCALED | (e + ADJT_BIAS): lambda is c 2^e
    // per tile and face (2 * axis + 1 for the + side), 64 cells of the face:
    double *fw;    // weighted difference to the upwind neighbour across the face (0: none)
    uint64_t *fo;  // contribution passed across it (ADJT_WAIT until the cell is solved, 0 bits: none)
    uint32_t *fl;  // the cell's level (ADJT_NOLEV until it is solved, 0: none)
    uint32_t *tag;           // last phase the tile was listed for
    uint32_t *list0, *list1;  // tiles of the current and the next phase
};
constexpr uint64_t ADJT_WAIT = ~0ull;
constexpr uint32_t ADJT_NOLEV = ~0u;
constexpr uint32_t ADJT_SCALED = 1u << 31;
constexpr int ADJT_BIAS = 1 << 14;

constexpr int ADJ_PACK = 16;
template <typename I> struct AdjPack {
    I v[ADJ_PACK];
    uint32_t first, n;
};

// Output gather: out[p] (accumulate ? += : =) sum over the m problems whose
// points start at base[k] of their gradient terms.
constexpr int ADJ_GATHER = 64;
struct AdjGather {
    double *out;
    int64_t n;
    int64_t base[ADJ_GATHER];
    uint32_t m, accumulate;
};

// The same for the tile sweep, by the problems' first tiles.
struct AdjTileGather {
    double *out;
    int64_t n0, n1, n2;
    int32_t t0, t1, t2;
    uint32_t tbase[ADJ_GATHER];
    const void *F[ADJ_GATHER];
    double h[ADJ_GATHER];
    uint32_t m, accumulate;
};

// Workspace carving for `total` points over n problems.
struct AdjLayout {
    size_t off_ctrl, off_inst, off_acc, off_cnt, off_code, off_list0, off_list1, total;
};

inline size_t adj_align(size_t x) { return (x + 255) / 256 * 256; }

inline AdjLayout adj_layout(int64_t n, uint64_t total)
{
    AdjLayout L;
    size_t o = 0;
    L.off_ctrl = o;
    o = adj_align(o + sizeof(AdjCtrl));
    L.off_inst = o;
    o = adj_align(o + sizeof(AdjInst) * (size_t)n);
    L.off_acc = o;
    o = adj_align(o + 8 * total);
    L.off_cnt = o;
    o = adj_align(o + 4 * total);
    L.off_code = o;
    o = adj_align(o + total);
    L.off_list0 = o;
    o = adj_align(o + 8 * total);
    L.off_list1 = o;
    o = adj_align(o + 8 * total);
    L.total = o;
    return L;
}

// The same for the tile sweep over nt tiles (36 bytes per cell of a tile).
struct AdjTileLayout {
    size_t off_ctrl, off_inst, off_head, off_row, off_u, off_c, off_lev, off_fw, off_fo, off_fl, off_tag, off_list0,
        off_list1, total;
};

inline AdjTileLayout adj_tile_layout(int64_t n, uint64_t nt)
{
    AdjTileLayout L;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = adj_align(o + bytes);
        return at;
    };
    L.off_ctrl = take(sizeof(AdjTileCtrl));
    L.off_inst = take(sizeof(AdjTileInst) * (size_t)n);
    L.off_head = take(64 * nt);
    L.off_row = take(8 * 64 * nt);
    L.off_u = take(8 * 512 * nt);
    L.off_c = take(8 * 512 * nt);
    L.off_lev = take(4 * 512 * nt);
    L.off_fw = take(8 * 384 * nt);
    L.off_fo = take(8 * 384 * nt);
    L.off_fl = take(4 * 384 * nt);
    L.off_tag = take(4 * nt);
    L.off_list0 = take(4 * nt);
    L.off_list1 = take(4 * nt);
    L.total = o;
    return L;
}

hipError_t launch_adjoint_tiles(const AdjTileParams &P, const AdjTileInst *insts, int64_t n, bool f64, hipStream_t s);
hipError_t launch_adjoint(const AdjParams &P, const AdjTileInst *insts, int64_t n, bool f64, hipStream_t s);

}  // namespace fmm
