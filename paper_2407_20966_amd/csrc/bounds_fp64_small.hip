// The 2D FP64 bounds kernel on grids of up to 16 x 16 and 32 x 32 nodes and on
// those within 48 x 48 that need no more than 2 x 3 nodes per thread, compiled
// without machine LICM, gfx950.
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

hipError_t launch_bounds_fp64_small(const BoundsArgs& a, int nodes_per_thread, hipStream_t stream) {
    return nodes_per_thread == 1 ? launch(bounds_fp64_2d<16, 16, 1, 1, 0>, kThreads, a, stream)
                                 : launch(bounds_fp64_2d<16, 16, 2, 2, 0>, kThreads, a, stream);
}

// A 33 x 41 grid leaves 41% of the 48 x 48 tile's work to nodes past the grid.
// With the threads split to fit it (17 x 14 of 2 x 3 nodes) a thread does six
// nodes instead of nine, in 119 VGPRs and 33 KB of LDS (tables of 16 states):
// four workgroups per CU instead of three.  2025 quads of 45 states: 57 against
// 75 us on 33 x 41 nodes, 55 against 71 on 36 x 36; 400 on 44 x 25: 25.6
// against 30.
bool bounds_fp64_fit(int nx, int ny) {
    return nx <= 48 && ny <= 48 && ((nx + 1) / 2) * ((ny + 2) / 3) <= kThreads;
}

hipError_t launch_bounds_fp64_fit(const BoundsArgs& a, hipStream_t stream) {
    if (!bounds_fp64_fit(a.nx, a.ny)) return hipErrorInvalidValue;
    return launch(bounds_fp64_2d<16, 16, 2, 3, 2, 48>, kThreads, a, stream);
}

}  // namespace kbl
