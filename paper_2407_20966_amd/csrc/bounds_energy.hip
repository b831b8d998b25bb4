// FP64 bounds with the energy envelopes of the per-state integrand (steps 1-3
// of the overview in Sec. 3.9, another reading of Sec. 3.6), gfx950: the method
// of bounds_fp64.hip with the energy integrand taken per state,
// E_min/max = sum_u M min/max_i g_i(u) (|u|^2/2 + theta_i delta/2), relaxed by
// (1 -+ r) like the distributions (eq. relaxed); rho and m as before.  The
// product g_i (h + c_i) has no log-domain shortcut, so the envelopes are kept
// in value space.  In 2D g_i is still separable in value space,
// g_i = exp(A_i[x]) exp(B_i[y]): both factors come from LDS tables built per
// chunk of states, and a pair costs one multiply for g, an add and a multiply
// for the integrand and four min/max.
//
// What bounds it: VALU issue, 7.5 ops per pair and a quarter more for the
// tables and the prologue.  The register allocator is asked for three waves
// per SIMD at 3 x 3 nodes per thread and for two at 4 x 4 (227 and 292 VGPRs
// without): a few values then wait in scratch outside the pair loop, and the
// other waves hide the table reads.  90000 quads of 80 states on a 48 x 48 grid:
// 4.44 ms, 4.85 with two waves; 40000 on 64 x 64: 3.37 ms, on 30 x 28: 1.05
// (3.42 and 1.08 before machine LICM was turned off here).
// Grids that need no more than 2 x 3 (within 48 x 48) or 3 x 4 nodes per thread
// get the threads split to fit them: 22500 quads of 45 states on 33 x 41 nodes
// take 619 us against 731 on the 3 x 3 tile, on 50 x 50 1.01 ms against 1.19.
// Visiting only the states that can be an extremum in a block of nodes, block
// by block as in bounds_cull_2d, does not pay here: it halves the pair work
// (36 of 80 states survive in 12 x 12 nodes), but the blocks near ties keep
// nearly all, and the other waves of the workgroup wait for theirs at the
// barriers of the tables (4.45 ms with sixteen blocks, 4.77 with 64).
#include "bounds_common.h"

namespace kbl {
namespace {

// FIT > 0: the threads are split to fit the grid, ceil(nx / TX) by ceil(ny / TY),
// with FIT x FIT tables; the threads left over repeat thread 0 with weight zero.
template <int BX, int BY, int TX, int TY, int FIT = 0>
__global__ __launch_bounds__(BX * BY)
__attribute__((amdgpu_waves_per_eu(TX * TY >= 12 ? 2 : TX * TY == 9 ? 3 : 4))) void bounds_fp64_2d_energy(BoundsArgs p) {
    constexpr int NT = BX * BY;
    constexpr int NXM = FIT ? FIT : BX * TX;
    constexpr int NYM = FIT ? FIT : BY * TY;
    constexpr int kTabStates = 32;
    static_assert(NT % 64 == 0 && NT <= kThreads, "workgroup must be 1-4 waves");
    __shared__ Coef sC[kMaxStates];
    __shared__ double sEA[kTabStates][NXM];
    __shared__ double sEB[kTabStates][NYM];
    __shared__ double sCs[kTabStates];        // theta delta / 2 per state
    __shared__ ExpPair sExp[256];
    __shared__ Red red;
    static_assert(NXM == NYM && NXM <= NT, "tables built by columns");

    const int tid = threadIdx.x;
    const int bx = FIT ? split_threads(p.nx, TX) : BX;
    const int by = FIT ? split_threads(p.ny, TY) : BY;
    const bool idle = FIT && tid >= bx * by;
    const int tx = idle ? 0 : tid % bx, ty = idle ? 0 : tid / bx;
    // table columns of this thread's nodes
    auto xcol = [&](int i) { return FIT ? split_column<FIT ? FIT : 1, TX>(tx + bx * i) : tx + bx * i; };
    auto ycol = [&](int j) { return FIT ? split_column<FIT ? FIT : 1, TY>(ty + by * j) : ty + by * j; };
    const double rm = 1.0 - p.r_fac, rp = 1.0 + p.r_fac;
    stage_exp_table<NT>(sExp);   // published by the prologue's barriers

    for (ElemRange er = xcd_range(p.n_elem, p.grid_blocks); er.e < er.end; er.e += er.step) {
        const int64_t e = er.e;
        const int64_t row0 = p.rowptr[e], row1 = p.rowptr[e + 1];
        if (row0 < 0 || row1 <= row0 || row1 > p.nnz) {
            if (tid == 0) store_nan<2>(p, e, KBL_ST_BAD_STENCIL);
            continue;
        }
        const int64_t S = (row1 - row0) * p.n_s;
        double box[4];
        const uint32_t flags = stencil_prologue<2, NT>(p, row0, S, red, sC, box);
        if (flags & (KBL_ST_BAD_STENCIL | KBL_ST_INADMISSIBLE)) {
            if (tid == 0) store_nan<2>(p, e, flags);
            continue;
        }
        const double lox = box[0], loy = box[2];
        const double hx = (box[1] - box[0]) / (double)(p.nx - 1);
        const double hy = (box[3] - box[2]) / (double)(p.ny - 1);
        double ux[TX], uy[TY], hux[TX], huy[TY];
#pragma unroll
        for (int i = 0; i < TX; ++i) {
            const int j = tx + bx * i;
            ux[i] = node_pos(lox, j < p.nx ? j : p.nx - 1, hx);
            hux[i] = 0.5 * ux[i] * ux[i];
        }
#pragma unroll
        for (int j = 0; j < TY; ++j) {
            const int jj = ty + by * j;
            uy[j] = node_pos(loy, jj < p.ny ? jj : p.ny - 1, hy);
            huy[j] = 0.5 * uy[j] * uy[j];
        }
        // no +-inf starting values: the stencil's first state sets the
        // envelopes (the empty asm gives the registers a defined value)
        double gn[TX][TY], gx[TX][TY], en[TX][TY], ex[TX][TY];
#pragma unroll
        for (int i = 0; i < TX; ++i)
#pragma unroll
            for (int j = 0; j < TY; ++j)
                asm volatile("" : "=v"(gn[i][j]), "=v"(gx[i][j]), "=v"(en[i][j]), "=v"(ex[i][j]));

        for (int64_t c0 = 0; c0 < S; c0 += kMaxStates) {
            const int cn = (int)((S - c0) < kMaxStates ? (S - c0) : kMaxStates);
            if (c0 > 0) stage_chunk<2, NT>(p, row0, c0, cn, sC);
            for (int t0 = 0; t0 < cn; t0 += kTabStates) {
                const int tn = (cn - t0) < kTabStates ? (cn - t0) : kTabStates;
                __syncthreads();
                {
                    // by columns: thread t fills node t % NXM of states
                    // t / NXM, t / NXM + NT / NXM, ...
                    constexpr int kPass = NT / NXM;
                    const int j = tid % NXM, sj = tid / NXM;
                    const double xj = node_pos(lox, j < p.nx ? j : p.nx - 1, hx);
                    const double yj = node_pos(loy, j < p.ny ? j : p.ny - 1, hy);
                    if (sj < kPass) {
                        for (int s = sj; s < tn; s += kPass) {
                            const Coef& c = sC[t0 + s];
                            const double dx = xj - c.ux;
                            sEA[s][j] = exp_tab(fma(c.nk * dx, dx, c.a), sExp);
                            const double dy = yj - c.uy;
                            sEB[s][j] = exp_tab((c.nk * dy) * dy, sExp);
                        }
                    }
                }
                for (int s = tid; s < tn; s += NT) sCs[s] = p.half_delta * (-0.5 / sC[t0 + s].nk);
                __syncthreads();
                int s0 = 0;
                if (c0 == 0 && t0 == 0) {
                    const double cs = sCs[0];
                    double ea[TX], hc[TX], eb[TY];
#pragma unroll
                    for (int i = 0; i < TX; ++i) {
                        ea[i] = sEA[0][xcol(i)];
                        hc[i] = hux[i] + cs;
                    }
#pragma unroll
                    for (int j = 0; j < TY; ++j) eb[j] = sEB[0][ycol(j)];
#pragma unroll
                    for (int i = 0; i < TX; ++i)
#pragma unroll
                        for (int j = 0; j < TY; ++j) {
                            const double g = ea[i] * eb[j];
                            const double eg = g * (hc[i] + huy[j]);
                            gn[i][j] = g;
                            gx[i][j] = g;
                            en[i][j] = eg;
                            ex[i][j] = eg;
                        }
                    s0 = 1;
                }
#pragma unroll 2
                for (int s = s0; s < tn; ++s) {
                    const double cs = sCs[s];
                    double ea[TX], hc[TX], eb[TY];
#pragma unroll
                    for (int i = 0; i < TX; ++i) {
                        ea[i] = sEA[s][xcol(i)];
                        hc[i] = hux[i] + cs;
                    }
#pragma unroll
                    for (int j = 0; j < TY; ++j) eb[j] = sEB[s][ycol(j)];
#pragma unroll
                    for (int i = 0; i < TX; ++i)
#pragma unroll
                        for (int j = 0; j < TY; ++j) {
                            const double g = ea[i] * eb[j];
                            const double eg = g * (hc[i] + huy[j]);
                            gn[i][j] = fmin(gn[i][j], g);
                            gx[i][j] = fmax(gx[i][j], g);
                            en[i][j] = fmin(en[i][j], eg);
                            ex[i][j] = fmax(ex[i][j], eg);
                        }
                }
            }
        }

        // separable contraction (M = wx wy; the sign of M u_k is the sign of
        // u_k): each node feeds per-row sums over y and per-column sums over
        // x, the moments are formed once per row and column, and (1 -+ r) is
        // applied to the sums
        double sr[2] = {0, 0}, se[2] = {0, 0}, mxs[2][2] = {{0, 0}, {0, 0}}, mys[2][2] = {{0, 0}, {0, 0}};
        double cn[TY], cx[TY];   // per column: sum over x of wx g_min, wx g_max
#pragma unroll
        for (int j = 0; j < TY; ++j) { cn[j] = 0.0; cx[j] = 0.0; }
#pragma unroll
        for (int i = 0; i < TX; ++i) {
            const int jx = tx + bx * i;
            if (idle || jx >= p.nx) continue;
            const double wx = hx * ((jx == 0 || jx == p.nx - 1) ? 0.5 : 1.0);
            double rn = 0.0, rx = 0.0, ren = 0.0, rex = 0.0;   // per row: sum over y of wy g, wy e
#pragma unroll
            for (int j = 0; j < TY; ++j) {
                const int jy = ty + by * j;
                if (jy >= p.ny) continue;
                const double wy = hy * ((jy == 0 || jy == p.ny - 1) ? 0.5 : 1.0);
                rn = fma(wy, gn[i][j], rn);
                rx = fma(wy, gx[i][j], rx);
                ren = fma(wy, en[i][j], ren);
                rex = fma(wy, ex[i][j], rex);
                cn[j] = fma(wx, gn[i][j], cn[j]);
                cx[j] = fma(wx, gx[i][j], cx[j]);
            }
            sr[0] = fma(wx, rn, sr[0]);
            sr[1] = fma(wx, rx, sr[1]);
            se[0] = fma(wx, ren, se[0]);
            se[1] = fma(wx, rex, se[1]);
            const double mu = wx * ux[i];
            const double neg = fmin(mu, 0.0), pos = fmax(mu, 0.0);
            mxs[0][0] = fma(neg, rx, mxs[0][0]);   // lower bound: u < 0 takes g_max
            mxs[0][1] = fma(pos, rn, mxs[0][1]);   //              u >= 0 takes g_min
            mxs[1][0] = fma(neg, rn, mxs[1][0]);   // upper bound: u < 0 takes g_min
            mxs[1][1] = fma(pos, rx, mxs[1][1]);   //              u >= 0 takes g_max
        }
#pragma unroll
        for (int j = 0; j < TY; ++j) {
            const int jy = ty + by * j;
            if (idle || jy >= p.ny) continue;
            const double wy = hy * ((jy == 0 || jy == p.ny - 1) ? 0.5 : 1.0);
            const double mu = wy * uy[j];
            const double neg = fmin(mu, 0.0), pos = fmax(mu, 0.0);
            mys[0][0] = fma(neg, cx[j], mys[0][0]);
            mys[0][1] = fma(pos, cn[j], mys[0][1]);
            mys[1][0] = fma(neg, cn[j], mys[1][0]);
            mys[1][1] = fma(pos, cx[j], mys[1][1]);
        }
        double part[8] = {rm * sr[0], rp * sr[1], rm * se[0], rp * se[1],
                          rp * mxs[0][0] + rm * mxs[0][1], rm * mxs[1][0] + rp * mxs[1][1],
                          rp * mys[0][0] + rm * mys[0][1], rm * mys[1][0] + rp * mys[1][1]};
        block_sum_t<NT, 8>(part, red);
        if (tid == 0) store_bounds<2>(p, e, part, flags);
    }
}

// 1D: no separability; one exp per (state, node) pair.
template <int NT, int T>
__global__ __launch_bounds__(NT) void bounds_fp64_1d_energy(BoundsArgs p) {
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
        double u[T], hu[T], gn[T], gx[T], en[T], ex[T];
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int j = tid + NT * i;
            u[i] = node_pos(lo, j < p.nx ? j : p.nx - 1, h);
            hu[i] = 0.5 * u[i] * u[i];
            gn[i] = kInf; gx[i] = -kInf; en[i] = kInf; ex[i] = -kInf;
        }
        for (int64_t c0 = 0; c0 < S; c0 += kMaxStates) {
            const int cn = (int)((S - c0) < kMaxStates ? (S - c0) : kMaxStates);
            if (c0 > 0) stage_chunk<1, NT>(p, row0, c0, cn, sC);
            for (int s = 0; s < cn; ++s) {
                const Coef c = sC[s];
                const double cs = p.half_delta * (-0.5 / c.nk);
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    const double d = u[i] - c.ux;
                    const double g = exp_tab(fma(c.nk * d, d, c.a), sExp);
                    const double eg = g * (hu[i] + cs);
                    gn[i] = fmin(gn[i], g);
                    gx[i] = fmax(gx[i], g);
                    en[i] = fmin(en[i], eg);
                    ex[i] = fmax(ex[i], eg);
                }
            }
        }
        double part[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int j = tid + NT * i;
            if (j >= p.nx) continue;
            const double M = h * ((j == 0 || j == p.nx - 1) ? 0.5 : 1.0);
            const double ftn = rm * gn[i], ftx = rp * gx[i];
            part[0] += M * ftn;
            part[1] += M * ftx;
            part[2] += M * (rm * en[i]);
            part[3] += M * (rp * ex[i]);
            if (u[i] < 0.0) { part[4] += M * u[i] * ftx; part[5] += M * u[i] * ftn; }
            else            { part[4] += M * u[i] * ftn; part[5] += M * u[i] * ftx; }
        }
        block_sum_t<NT, 6>(part, red);
        if (tid == 0) store_bounds<1>(p, e, part, flags);
    }
}

template <typename K>
hipError_t launch(K kernel, int threads, const BoundsArgs& a, hipStream_t stream) {
    hipLaunchKernelGGL(kernel, dim3(bounds_grid(a)), dim3(threads), 0, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_bounds_fp64_energy(const BoundsArgs& a, int dim, hipStream_t stream) {
    if (a.n_elem == 0) return hipSuccess;
    if (dim == 2) {
        const int n = a.nx > a.ny ? a.nx : a.ny;
        if (n <= 16) return launch(bounds_fp64_2d_energy<16, 16, 1, 1>, 256, a, stream);
        if (n <= 32) return launch(bounds_fp64_2d_energy<16, 16, 2, 2>, 256, a, stream);
        if (n <= 48 && tile_fits_grid<2, 3>(a))
            return launch(bounds_fp64_2d_energy<16, 16, 2, 3, 48>, 256, a, stream);
        if (n <= 48) return launch(bounds_fp64_2d_energy<16, 16, 3, 3>, 256, a, stream);
        if (n <= 64 && tile_fits_grid<3, 4>(a))
            return launch(bounds_fp64_2d_energy<16, 16, 3, 4, 64>, 256, a, stream);
        if (n <= 64) return launch(bounds_fp64_2d_energy<16, 16, 4, 4>, 256, a, stream);
        return hipErrorInvalidValue;
    }
    if (a.nx <= 64) return launch(bounds_fp64_1d_energy<64, 1>, 64, a, stream);
    if (a.nx <= 256) return launch(bounds_fp64_1d_energy<256, 1>, kThreads, a, stream);
    if (a.nx <= 512) return launch(bounds_fp64_1d_energy<256, 2>, kThreads, a, stream);
    if (a.nx <= 1024) return launch(bounds_fp64_1d_energy<256, 4>, kThreads, a, stream);
    if (a.nx <= 2048) return launch(bounds_fp64_1d_energy<256, 8>, kThreads, a, stream);
    if (a.nx <= 4096) return launch(bounds_fp64_1d_energy<256, 16>, kThreads, a, stream);
    return hipErrorInvalidValue;
}

}  // namespace kbl
