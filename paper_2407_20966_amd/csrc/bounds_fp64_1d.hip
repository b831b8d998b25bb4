// FP64 kinetic bounds over a one-dimensional velocity grid (steps 1-3 of the
// overview in Sec. 3.9), gfx950: the method of bounds_fp64.hip without the
// separable tables.
#include "bounds_1d.h"

namespace kbl {
namespace {

// One workgroup per element; the nodes go in rounds of NT T (thread t owns
// nodes t + NT i of a round, with CULL a wave 64 T consecutive ones).
// What bounds it: VALU issue, 8 ops per (state, node) and 77 per node for the
// four exps and the moments.  Two nodes per thread and round and at most 96
// VGPRs keep five waves on a SIMD to cover the prologue, the exp table reads
// and the barriers: 20000 stencils of 12 states take 253 us with 2048 nodes,
// 9 states 142 with 1000 (290 and 171 with all of a thread's nodes at once, in up
// to 168 VGPRs; four nodes per round, four waves: 254, 145); 30000 with 200 nodes
// take 125 us against 144.  Up to 512 nodes there is one round in any case (the
// rule below).
// CULL (grids beyond 512 nodes, ten states and more): a wave's 128 nodes of a
// round are a block over which five of 12 or seven of 18 states can be an
// extremum.  Lane = (round, state) bounds up to four rounds at once, the ballot is
// the mask of states to visit.  2048 nodes: 12 states 205 us against 253, 18
// states 234 against 315; 700 nodes, 12 states 137 against 153; where states
// tie up to rounding all are visited in the plain loop, of equal states one is
// (20000 stencils of 12 on 1100 nodes: 133 us, 195 with all, 254 before the cull).
// The 1D solver's stencils of 6 to 12 states gain nothing by it.
template <int NT, int T, bool CULL, int WAVES>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WAVES)))
void bounds_fp64_1d(BoundsArgs p) {
    __shared__ Coef sC[kMaxStates];
    __shared__ ExpPair sExp[256];
    __shared__ Red red;
    const int tid = threadIdx.x;
    const double rm = 1.0 - p.r_fac, rp = 1.0 + p.r_fac;
    stage_exp_table<NT>(sExp);   // published by the prologue's barriers
    for (ElemRange er = xcd_range(p.n_elem, p.grid_blocks); er.e < er.end; er.e += er.step) {
        const int64_t e = er.e;
        const int64_t row0 = p.rowptr[e], row1 = p.rowptr[e + 1];
        if (row0 < 0 || row1 <= row0 || row1 > p.nnz) {
            if (tid == 0) store_nan<1>(p, e, KBL_ST_BAD_STENCIL);
            continue;
        }
        const int64_t S = (row1 - row0) * p.n_s;
        double box[4];
        const uint32_t flags = stencil_prologue<1, NT>(p, row0, S, red, sC, box);
        if (flags & (KBL_ST_BAD_STENCIL | KBL_ST_INADMISSIBLE)) {
            if (tid == 0) store_nan<1>(p, e, flags);
            continue;
        }
        const double lo = box[0];
        const double h = (box[1] - box[0]) / (double)(p.nx - 1);
        Sums1D sum1;
        if (S <= kMaxStates) {
            const int rounds = (p.nx + NT * T - 1) / (NT * T);
            if (CULL && S >= 10 && S <= 64 && S * rounds >= 24) {
                // the waves take consecutive runs of nodes and visit the
                // states that can be an extremum there
                const int lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
                const int lg = S <= 16 ? 4 : S <= 32 ? 5 : 6;
                unsigned long long bits = 0;
                for (int r = 0; r < rounds; ++r) {
                    const int sub = r & ((64 >> lg) - 1);
                    if (sub == 0) bits = cull_1d<NT, T>(p, sC, (int)S, lo, h, r, lg);
                    const unsigned long long m = (bits >> (sub << lg)) & (~0ull >> (64 - (1 << lg)));
                    if (m == 0) break;         // past the grid
                    const int j0 = r * NT * T + wid * 64 * T + lane;
                    Env1D<T> env;
                    // (nearly) tied states: all of them in the plain loop
                    if (8 * __popcll(m) > 7 * (int)S) env.fold(p, sC, (int)S, lo, h, j0, 64, true);
                    else env.fold_mask(p, sC, m, lo, h, j0, 64);
                    env.contract(p, lo, h, j0, 64, sExp, sum1);
                }
            } else {
                for (int j0 = 0; j0 < p.nx; j0 += NT * T) {
                    Env1D<T> env;
                    env.fold(p, sC, (int)S, lo, h, j0 + tid, NT, true);
                    env.contract(p, lo, h, j0 + tid, NT, sExp, sum1);
                }
            }
        } else {
            // chunks of states, staged again in every round; one node per
            // thread keeps the registers of the staging's logs out of the
            // way of the branch above
            for (int j0 = 0; j0 < p.nx; j0 += NT) {
                Env1D<1> env;
                for (int64_t c0 = 0; c0 < S; c0 += kMaxStates) {
                    const int cn = (int)((S - c0) < kMaxStates ? (S - c0) : kMaxStates);
                    stage_chunk<1, NT>(p, row0, c0, cn, sC);
                    env.fold(p, sC, cn, lo, h, j0 + tid, NT, c0 == 0);
                }
                env.contract(p, lo, h, j0 + tid, NT, sExp, sum1);
            }
        }
        double part[8];
        sum1.parts(rm, rp, part);
        const double sum = block_sum8<NT>(part, red);
        if (tid < 6) store_bound_value<1>(p, e, tid, sum, flags);
    }
}

// Stencils beyond the staged states: all of a thread's nodes at once, so that every
// chunk of states is staged once per element (in rounds of one node per thread
// each chunk's logs are formed again in every round).  1000 stencils of 300
// states: 172 us with 2048 nodes (296 in rounds), 54 with 300 (80), 29 with 40 (32).
// Two waves per SIMD for eight nodes per thread: 186 us on 2048 nodes with three.
template <int NT, int T>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(T < 8 ? 3 : T == 8 ? 2 : 1)))
void bounds_fp64_1d_chunks(BoundsArgs p) {
    __shared__ Coef sC[kMaxStates];
    __shared__ ExpPair sExp[256];
    __shared__ Red red;
    const int tid = threadIdx.x;
    const double rm = 1.0 - p.r_fac, rp = 1.0 + p.r_fac;
    stage_exp_table<NT>(sExp);   // published by the prologue's barriers
    for (ElemRange er = xcd_range(p.n_elem, p.grid_blocks); er.e < er.end; er.e += er.step) {
        const int64_t e = er.e;
        const int64_t row0 = p.rowptr[e], row1 = p.rowptr[e + 1];
        if (row0 < 0 || row1 <= row0 || row1 > p.nnz) {
            if (tid == 0) store_nan<1>(p, e, KBL_ST_BAD_STENCIL);
            continue;
        }
        const int64_t S = (row1 - row0) * p.n_s;
        double box[4];
        const uint32_t flags = stencil_prologue<1, NT>(p, row0, S, red, sC, box);
        if (flags & (KBL_ST_BAD_STENCIL | KBL_ST_INADMISSIBLE)) {
            if (tid == 0) store_nan<1>(p, e, flags);
            continue;
        }
        const double lo = box[0];
        const double h = (box[1] - box[0]) / (double)(p.nx - 1);
        Env1D<T> env;
        for (int64_t c0 = 0; c0 < S; c0 += kMaxStates) {
            const int cn = (int)((S - c0) < kMaxStates ? (S - c0) : kMaxStates);
            if (c0 > 0) stage_chunk<1, NT>(p, row0, c0, cn, sC);
            env.fold(p, sC, cn, lo, h, tid, NT, c0 == 0);
        }
        Sums1D sum1;
        env.contract(p, lo, h, tid, NT, sExp, sum1);
        double part[8];
        sum1.parts(rm, rp, part);
        const double sum = block_sum8<NT>(part, red);
        if (tid < 6) store_bound_value<1>(p, e, tid, sum, flags);
    }
}

template <int NT, int T>
hipError_t launch_1d_chunks(const BoundsArgs& a, hipStream_t stream) {
    hipLaunchKernelGGL((bounds_fp64_1d_chunks<NT, T>), dim3(bounds_grid(a)), dim3(NT), 0, stream, a);
    return hipGetLastError();
}

template <int NT, int T, bool CULL = false, int WAVES = 5>
hipError_t launch_1d(const BoundsArgs& a, hipStream_t stream) {
    hipLaunchKernelGGL((bounds_fp64_1d<NT, T, CULL, WAVES>), dim3(bounds_grid(a)), dim3(NT), 0, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_bounds_fp64_1d(const BoundsArgs& a, hipStream_t stream) {
    // rows of both kinds take the rounds above, chunk by chunk where they must
    if (!states_at_most(a, kMaxStates)) {
        if (a.nx <= 64) return launch_1d_chunks<64, 1>(a, stream);
        if (a.nx <= 256) return launch_1d_chunks<256, 1>(a, stream);
        if (a.nx <= 512) return launch_1d_chunks<256, 2>(a, stream);
        if (a.nx <= 1024) return launch_1d_chunks<256, 4>(a, stream);
        if (a.nx <= 2048) return launch_1d_chunks<256, 8>(a, stream);
        return launch_1d_chunks<256, 16>(a, stream);
    }
    if (a.nx <= 64) return launch_1d<64, 1>(a, stream);
    if (a.nx <= 256) return launch_1d<256, 1>(a, stream);
    // Meshes of up to three workgroups per CU or so are bound by the latency of one
    // workgroup's rounds, not by the waves in flight: all nodes in one round there, in
    // the registers of fewer waves.  Up to 512 nodes, 3 to 18 states: 7.1-8.1 us at
    // 500 to 700 elements against 7.2-8.7 in the five-wave form; from 768 on 128
    // threads with four nodes each, 7.2-8.7 at 1000 elements against 7.9-9.8, 75 us at
    // 20000 elements of 6 states against 93.
    const bool few = a.n_elem < 768;
    if (a.nx <= 512)
        return few ? launch_1d<256, 2, false, 3>(a, stream) : launch_1d<128, 4, false, 3>(a, stream);
    // Up to 1024 nodes likewise, unless the cull below is worth more: 12 states
    // 6.8-8.4 us at 32 to 500 elements against 7.7-9.4 with it, 18 states 8.9 and
    // 9.0-9.6, 30 states 10.8 and 10.2; at 850 elements 10 states 10.3 and 11.7, 12
    // states 10.8 and 10.3-11.7.
    if (a.nx <= 1024 && (few ? !states_at_least(a, 18)
                             : a.n_elem < 1024 && !states_at_least(a, 12)))
        return launch_1d<256, 4, false, 4>(a, stream);
    // a pass of the cull costs a wave about 80 ops, a state left out 16 per
    // round of 512 nodes: from two rounds and a dozen states on (below that the
    // plain kernel is 3-5% faster)
    if (states_at_least(a, 10)) return launch_1d<256, 2, true>(a, stream);
    return launch_1d<256, 2>(a, stream);
}

}  // namespace kbl
