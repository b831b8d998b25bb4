// The 2D FP64 bounds kernel on grids of up to 16 x 16 and 32 x 32 nodes and on
// larger ones that need no more than 2 x 3 (within 48 x 48) or 3 x 4 nodes per
// thread, compiled without machine LICM, gfx950.
//
// What bounds it: VALU issue, with the prologue's logs and the contraction's
// exps a large part beside one or four nodes per thread.  Machine LICM hoists
// the constants of both out of the loop over elements and keeps them in
// registers throughout: without it the kernel fits five and four waves per SIMD
// (89 and 121 VGPRs) instead of four and three (117 and 149).  90000 quads
// of 45 states on 16 x 16 nodes take 720 us against 790, on 24 x 24 1.43 ms
// against 1.58, 4900 of 80 states on 32 x 30 140 us against 145.  The larger
// tiles keep it: 64 x 64 on LDS tables runs 3% slower without.
#include "bounds_2d.h"

namespace kbl {

// Grids between 16 and 32 nodes likewise, with one x node and two or three y
// nodes per thread where 256 threads cover them so: 2025 quads of 45 states on 20
// x 20 nodes 27 us against 38 with 2 x 2, on 24 x 24 34 against 38; 62500 on 20 x 20
// 671 against 989, on 24 x 24 840 against 1004.
hipError_t launch_bounds_fp64_small(const BoundsArgs& a, int nodes_per_thread, hipStream_t stream) {
    if (nodes_per_thread == 1) return launch(bounds_fp64_2d<16, 16, 1, 1, 0>, kThreads, a, stream);
    if (tile_fits_grid<1, 2>(a))
        return launch(bounds_fp64_2d<16, 16, 1, 2, 0, 32>, kThreads, a, stream);
    if (tile_fits_grid<1, 3>(a))
        return launch(bounds_fp64_2d<16, 16, 1, 3, 0, 32>, kThreads, a, stream);
    return launch(bounds_fp64_2d<16, 16, 2, 2, 0>, kThreads, a, stream);
}

// A 33 x 41 grid leaves 41% of the 48 x 48 tile's work to nodes past the grid.
// With the threads split to fit it (17 x 14 of 2 x 3 nodes) a thread does six
// nodes instead of nine, in 119 VGPRs and 33 KB of LDS (tables of 16 states):
// four workgroups per CU instead of three.  2025 quads of 45 states: 57 against
// 75 us on 33 x 41 nodes, 55 against 71 on 36 x 36; 400 on 44 x 25: 25.6
// against 30.  Likewise beyond 48 nodes with 3 x 4 nodes per thread instead of
// 4 x 4: 2025 quads of 45 states on 50 x 50 102 us against 112.
bool bounds_fp64_fit(const BoundsArgs& a) {
    return a.nx <= 48 && a.ny <= 48 ? tile_fits_grid<2, 3>(a)
                                    : a.nx <= 64 && a.ny <= 64 && tile_fits_grid<3, 4>(a);
}

hipError_t launch_bounds_fp64_fit(const BoundsArgs& a, hipStream_t stream) {
    if (!bounds_fp64_fit(a)) return hipErrorInvalidValue;
    if (a.nx <= 48 && a.ny <= 48)
        return launch(bounds_fp64_2d<16, 16, 2, 3, 2, 48>, kThreads, a, stream);
    return launch(bounds_fp64_2d<16, 16, 3, 4, 2, 64>, kThreads, a, stream);
}

}  // namespace kbl
