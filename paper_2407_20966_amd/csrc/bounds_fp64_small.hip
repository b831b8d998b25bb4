// The 2D FP64 bounds kernel on grids of up to 16 x 16 and 32 x 32 nodes,
// compiled without machine LICM, gfx950.
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

}  // namespace kbl
