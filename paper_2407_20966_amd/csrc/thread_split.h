// How the 256 threads of a workgroup are split to fit a 2D velocity grid: TX x TY
// nodes per thread, ceil(nx / TX) x ceil(ny / TY) threads, thread t owning nodes
// t + threads * i of a direction.  Plain constexpr functions: host code, device
// code and the tests share them.
#pragma once

namespace kbl {

// Threads along a direction of n nodes with T nodes each.
constexpr int split_threads(int n, int T) { return (n + T - 1) / T; }

// Whether 256 threads with TX x TY nodes each cover nx x ny nodes.
template <int TX, int TY>
constexpr bool split_fits(int nx, int ny) {
    return split_threads(nx, TX) * split_threads(ny, TY) <= 256;
}

// Column of a FIT-wide table for a node of such a thread.  Where T does not
// divide FIT the last threads' nodes reach past the widest grid (64 nodes by
// three: 22 threads, 66 nodes); those read the last column, and their results
// are not used.
template <int FIT, int T>
constexpr int split_column(int node) {
    return FIT % T == 0 || node < FIT ? node : FIT - 1;
}

}  // namespace kbl
