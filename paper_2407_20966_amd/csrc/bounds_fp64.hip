// FP64 kinetic bounds (steps 1-3 of the overview in Sec. 3.9), gfx950.
//
// One workgroup (1-4 wave64) owns one element at a time.
//  1. Prologue: every stencil state (every node of every element of the CSR
//     row) is read once, checked for admissibility (Assumption (i) of Sec. 4)
//     and turned into the coefficients of its log-Maxwellian
//       q_i(u) = ln rho_i - (d/2) ln(2 pi theta_i) - |u - U_i|^2 / (2 theta_i),
//     which are staged in LDS; in STENCIL mode the velocity box of
//     eq. truncdomain is reduced on the way.
//  2. Hot loop over the states: q_i is separable on the Cartesian velocity
//     grid, q_i = A_i[jx] + B_i[jy].  Each thread evaluates A (and
//     A + ln(theta delta / 2)) for its x nodes and B for its y nodes, then
//     spends two adds and four min/max per (state, node) pair.  Because exp is
//     monotone, min_i g_i = exp(min_i q_i) (eq. fminmax), and likewise for the
//     internal part g_I = (theta delta / 2) g (Sec. 3.6): four running extrema
//     per node stay in registers and only four exp per node are taken at the
//     end.  (Tile variants read B, or A and B, from LDS tables instead.)
//  3. Relaxation (eq. relaxed), trapezoid weights (Sec. 3.7) and the moment
//     contraction (eq. rhobounds, Ebounds, mmbounds, mpbounds) are done per
//     node, then reduced across the workgroup in a fixed order (bitwise
//     deterministic), floored (Sec. 3.8) and stored.
// Each thread owns a TX x TY tile of velocity nodes, strided by 16 so that
// the LDS table reads of a wave are contiguous or broadcast.  Tile modes:
// BTAB = 0 computes A and B per state in registers; 1 reads B from a table
// built per chunk of states; 2 reads A, A + ln(theta delta / 2) and B from
// such tables (per state: a few LDS reads instead of 4 TX + 3 TY VALU ops).
// Inputs are validated before the hot loop, which therefore never sees a NaN
// (only finite values and -inf when delta = 0).
#include "bounds_2d.h"

namespace kbl {
namespace {

// 2D tile configurations: (BX, BY, TX, TY, BTAB) covers nx <= BX*TX, ny <= BY*TY.
struct Tile2D {
    int bx, by, tx, ty, btab;
    hipError_t (*fn)(const BoundsArgs&, hipStream_t);
};

template <int BX, int BY, int TX, int TY, int BTAB>
hipError_t launch_2d(const BoundsArgs& a, hipStream_t stream) {
    return launch(bounds_fp64_2d<BX, BY, TX, TY, BTAB>, BX * BY, a, stream);
}

// the tiles compiled in bounds_fp64_small.hip
template <>
hipError_t launch_2d<16, 16, 1, 1, 0>(const BoundsArgs& a, hipStream_t stream) {
    return launch_bounds_fp64_small(a, 1, stream);
}
template <>
hipError_t launch_2d<16, 16, 2, 2, 0>(const BoundsArgs& a, hipStream_t stream) {
    return launch_bounds_fp64_small(a, 2, stream);
}

// the table tiles, split to fit grids that leave a third or a quarter of them
// unused (a grid within 48 x 48 keeps the 64 x 64 tile if that was asked for)
template <>
hipError_t launch_2d<16, 16, 3, 3, 2>(const BoundsArgs& a, hipStream_t stream) {
    if (bounds_fp64_fit(a)) return launch_bounds_fp64_fit(a, stream);
    return launch(bounds_fp64_2d<16, 16, 3, 3, 2>, kThreads, a, stream);
}
template <>
hipError_t launch_2d<16, 16, 4, 4, 2>(const BoundsArgs& a, hipStream_t stream) {
    if ((a.nx > 48 || a.ny > 48) && bounds_fp64_fit(a)) return launch_bounds_fp64_fit(a, stream);
    return launch(bounds_fp64_2d<16, 16, 4, 4, 2>, kThreads, a, stream);
}

// mode 3: the kernel that culls states block by block
template <>
hipError_t launch_2d<16, 16, 4, 4, 3>(const BoundsArgs& a, hipStream_t stream) {
    return launch_bounds_cull_2d(a, stream);
}

#define KBL_TILE(BX, BY, TX, TY, M) {BX, BY, TX, TY, M, launch_2d<BX, BY, TX, TY, M>}
constexpr Tile2D kTiles2D[] = {
    KBL_TILE(16, 16, 1, 1, 0),   // 0: n <= 16
    KBL_TILE(16, 16, 2, 2, 0),   // 1: n <= 32
    KBL_TILE(16, 16, 3, 3, 0),   // 2: n <= 48
    KBL_TILE(16, 16, 3, 3, 1),   // 3: n <= 48, B from LDS
    KBL_TILE(16, 8, 3, 6, 0),    // 4: n <= 48, two waves
    KBL_TILE(16, 16, 4, 4, 0),   // 5: n <= 64
    KBL_TILE(16, 16, 4, 4, 1),   // 6: n <= 64, B from LDS
    KBL_TILE(32, 8, 2, 8, 1),    // 7: n <= 64, B from LDS
    KBL_TILE(16, 16, 2, 4, 0),   // 8: nx <= 32, ny <= 64
    KBL_TILE(16, 16, 4, 2, 0),   // 9: nx <= 64, ny <= 32
    KBL_TILE(16, 16, 2, 2, 2),   // 10: n <= 32, A and B from LDS
    KBL_TILE(16, 16, 3, 3, 2),   // 11: n <= 48, A and B from LDS
    KBL_TILE(16, 16, 4, 4, 2),   // 12: n <= 64, A and B from LDS
    KBL_TILE(16, 8, 3, 6, 2),    // 13: n <= 48, two waves, A and B from LDS
    KBL_TILE(16, 16, 4, 4, 3),   // 14: n <= 64, states culled block by block
};
#undef KBL_TILE
constexpr int kCullTile2 = 14;
constexpr int kNumTiles2D = sizeof(kTiles2D) / sizeof(kTiles2D[0]);

// Defaults from a measured sweep: with A, A + l and B read from LDS tables
// the inner loop is the pair work alone (tiles 11 and 12); kbl_autotune_bounds
// may still pick another tile or a persistent grid for a given shape.
int default_tile_2d(int nx, int ny) {
    const int n = nx > ny ? nx : ny;
    if (n <= 16) return 0;
    if (n <= 32) return 1;
    if (n <= 48) return 11;
    return 12;
}

// Whether the culling kernel (tile 14) is the default.  It walks one element
// per wave, so it needs a few thousand elements to fill the chip, and its
// gain grows with the grid (blocks become small against the width of the
// Maxwellians) and with the stencil.  Times of the other default over those of
// the culling kernel, quads of 20, 45 and 80 states:
//  - grids beyond 48 nodes: 0.94-1.11 at 2025 elements, 1.12-1.26 at 3025;
//  - beyond 32 nodes, at most eight passes, no fit to the grid (40 x 40):
//    1.04-1.07 at 2500, 1.17 at 3600, 1.3-1.5 at 40000;
//  - beyond 32 nodes with a fit (36 x 41) or more passes (48 x 48): 0.8-0.97 and
//    0.94-1.02 with 20 states; with 45 and more 0.9-1.0 at 6400 elements,
//    1.0-1.1 at 10000, 1.16-1.22 at 40000;
//  - up to 32 nodes (32 x 30): 0.87-0.95 with 20 states, with 45 and more 1.0 at
//    6400, 1.02-1.15 from 10000 on; up to 28 nodes 0.86-1.01 (triangles of 84
//    states 1.04-1.2); below 0.9 on those that one to three nodes per thread
//    cover (30 x 16).
// Node stencils (n_s = 1, of 48 states with the same values on both sides of a
// face) have longer lists: 0.9-0.99 up to 16000, 0.95-1.05 beyond.
// Stencils beyond the states it stages cannot be culled: 130 states 0.61-0.86
// (30 x 30 to 64 x 64 nodes, 4096 and 16384 elements), 180 to 320 states 0.60-0.89;
// 128 states 0.97-1.43.  Where rows of 110 and 140 alternate 0.78-1.0: the mean
// is all that is known here.
// With a handful of states there is little to leave out: 4 to 9 states 0.87-1.0 from
// 3000 to 6400 elements (40 x 40 and 64 x 64 nodes), 13 and more 0.96-1.1; from 10000
// on 0.98-1.16 with 4 to 9 too.
bool cull_pays(const BoundsArgs& a) {
    if (!bounds_cull_fits(a) || !states_at_most(a, kCullCap)) return false;
    const int n = a.nx > a.ny ? a.nx : a.ny;
    if (n <= 24 || a.n_elem < 3000) return false;
    if (a.n_elem < 8192 && !states_at_least(a, 12)) return false;
    if (n > 48) return true;
    if (n <= 32 && tile_fits_grid<1, 3>(a)) return false;
    const int hw = (a.nx + 15) / 16, hh = (a.ny + 15) / 16;
    const int blocks = ((a.nx + 2 * hw - 1) / (2 * hw)) * ((a.ny + 2 * hh - 1) / (2 * hh));
    if (n > 32 && blocks <= 8 * (64 / (hw * hh)) && !bounds_fp64_fit(a)) return true;
    if (n <= 28) return a.n_elem >= 32768 && states_at_least(a, 64);
    return a.n_s > 1 && states_at_least(a, 40) && a.n_elem >= 8192;
}

}  // namespace

int bounds_tile_count_2d() { return kNumTiles2D; }

int bounds_default_tile_2d(const BoundsArgs& a, int64_t* blocks) {
    *blocks = a.grid_blocks;
    if (!cull_pays(a)) return default_tile_2d(a.nx, a.ny);
    // one element per wave on small meshes (less of a tail)
    if (a.grid_blocks == -2 && a.n_elem < 65536) *blocks = 0;
    return kCullTile2;
}

bool bounds_tile_fits_2d(int tile, const BoundsArgs& a) {
    if (tile < 0 || tile >= kNumTiles2D) return false;
    const Tile2D& t = kTiles2D[tile];
    return a.nx <= t.bx * t.tx && a.ny <= t.by * t.ty && (tile != kCullTile2 || bounds_cull_fits(a));
}

hipError_t launch_bounds_fp64(const BoundsArgs& a, int dim, hipStream_t stream, int tile) {
    if (a.n_elem == 0) return hipSuccess;
    if (dim == 2) {
        if (!bounds_tile_fits_2d(tile, a)) return hipErrorInvalidValue;
        return kTiles2D[tile].fn(a, stream);
    }
    return launch_bounds_fp64_1d(a, stream);
}

}  // namespace kbl
