// Every table read of the kernels whose threads are split to fit the grid
// (csrc/thread_split.h), for every grid they accept: columns stay inside the
// table, each node has exactly one thread and reads its own column.
#include <cstdio>
#include <vector>

#include "thread_split.h"

static long bad = 0;

template <int FIT, int T>
static void direction(int n) {
    std::vector<int> seen(n, 0);
    const int threads = kbl::split_threads(n, T);
    for (int t = 0; t < threads; ++t)
        for (int i = 0; i < T; ++i) {
            const int node = t + threads * i, col = kbl::split_column<FIT, T>(node);
            if (col < 0 || col >= FIT || (node < n && col != node)) {
                std::printf("%d nodes by %d in a table of %d: node %d reads column %d\n", n, T, FIT,
                            node, col);
                ++bad;
            }
            if (node < n) ++seen[node];
        }
    for (int j = 0; j < n; ++j)
        if (seen[j] != 1) ++bad;
}

template <int FIT, int TX, int TY>
static int tile() {
    int grids = 0;
    for (int nx = 2; nx <= FIT; ++nx)
        for (int ny = 2; ny <= FIT; ++ny) {
            if (!kbl::split_fits<TX, TY>(nx, ny)) continue;
            direction<FIT, TX>(nx);
            direction<FIT, TY>(ny);
            ++grids;
        }
    return grids;
}

int main() {
    const int grids = tile<48, 2, 3>() + tile<64, 3, 4>();
    std::printf("%d grids, %ld bad reads\n", grids, bad);
    return bad || grids < 1000 ? 1 : 0;
}
