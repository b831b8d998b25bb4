// The 2D FP64 bounds kernel that evaluates every stencil state at every node
// (the method at the head of bounds_fp64.hip), for its translation units.
#pragma once

#include "bounds_common.h"

namespace kbl {
namespace {

// ---------------------------------------------------------------- 2D kernel
// BX x BY threads; thread (tx, ty) owns velocity nodes (tx + BX i, ty + BY j),
// i < TX, j < TY.  BTAB = 1 reads B (and BTAB = 2 also A, A + l) from LDS
// tables built per sub-chunk of kTabStates states (fewer VALU ops, more LDS
// traffic and barriers).  FIT > 0: the threads are split to fit the grid, bx =
// ceil(nx / TX) by by = ceil(ny / TY), with FIT x FIT tables; the threads left
// over repeat thread 0 with weight zero.
template <int BX, int BY, int TX, int TY, int BTAB, int FIT = 0>
__global__ __launch_bounds__(BX * BY)
__attribute__((amdgpu_waves_per_eu(FIT ? (TX * TY <= 3 ? 5 : TX * TY <= 6 ? 4 : 2) : BTAB == 2 ? (TX * TY <= 9 ? 3 : 2) : 1))) void bounds_fp64_2d(BoundsArgs p) {
    constexpr int NT = BX * BY;
    constexpr int NXM = FIT ? FIT : BX * TX;
    constexpr int NYM = FIT ? FIT : BY * TY;
    constexpr int kTabStates = FIT ? 16 : 32;
    static_assert(NT % 64 == 0 && NT <= kThreads, "workgroup must be 1-4 waves");
    static_assert(BTAB == 0 || (NXM == NYM && NYM <= NT), "table tiles are square");
    __shared__ Coef sC[kMaxStates];
    __shared__ double sB[BTAB ? kTabStates : 1][BTAB ? NYM : 1];
    // BTAB = 2: A and A + l tables too (row 2s: A, row 2s+1: A + l)
    __shared__ double sA[BTAB == 2 ? 2 * kTabStates : 1][BTAB == 2 ? NXM : 1];
    __shared__ ExpPair sExp[256];
    __shared__ Red red;

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

        // node coordinates (clamped into the grid for the ragged tail)
        double ux[TX], uy[TY];
#pragma unroll
        for (int i = 0; i < TX; ++i) {
            const int j = tx + bx * i;
            ux[i] = node_pos(lox, j < p.nx ? j : p.nx - 1, hx);
        }
#pragma unroll
        for (int j = 0; j < TY; ++j) {
            const int jj = ty + by * j;
            uy[j] = node_pos(loy, jj < p.ny ? jj : p.ny - 1, hy);
        }

        // No +-inf starting values (two moves per accumulator): the
        // stencil's first state writes the envelopes in the peeled first
        // step of the hot loop; the empty asm gives the registers a defined
        // value until then.
        double qtn[TX][TY], qtx[TX][TY], qin[TX][TY], qix[TX][TY];
#pragma unroll
        for (int i = 0; i < TX; ++i)
#pragma unroll
            for (int j = 0; j < TY; ++j)
                asm volatile("" : "=v"(qtn[i][j]), "=v"(qtx[i][j]), "=v"(qin[i][j]), "=v"(qix[i][j]));

        for (int64_t c0 = 0; c0 < S; c0 += kMaxStates) {
            const int cn = (int)((S - c0) < kMaxStates ? (S - c0) : kMaxStates);
            if (c0 > 0) stage_chunk<2, NT>(p, row0, c0, cn, sC);
            for (int t0 = 0; t0 < cn; t0 += (BTAB ? kTabStates : kMaxStates)) {
                const int tn = BTAB ? ((cn - t0) < kTabStates ? (cn - t0) : kTabStates) : cn;
                if (BTAB) {
                    // Table columns: thread t fills node t % NYM of states
                    // t / NYM, t / NYM + NT / NYM, ... (one node coordinate
                    // per thread, no index arithmetic per entry).  The thread
                    // index goes through an empty asm statement so that the
                    // column and its coordinate are formed here, not kept
                    // live across the hot loop.
                    int ot = tid;
                    asm volatile("" : "+v"(ot));
                    const int j = ot % NYM, sj = ot / NYM;
                    const double yj = node_pos(loy, j < p.ny ? j : p.ny - 1, hy);
                    const double xj = node_pos(lox, j < p.nx ? j : p.nx - 1, hx);
                    __syncthreads();
                    if (sj < NT / NYM) {
                        // fully unrolled (LDS offsets become immediates)
                        constexpr int kPass = NT / NYM;
#pragma unroll
                        for (int k = 0; k < (kTabStates + kPass - 1) / kPass; ++k) {
                            const int s = sj + kPass * k;
                            if (s >= tn) break;
                            const Coef c = sC[t0 + s];
                            const double d = yj - c.uy;
                            sB[s][j] = (c.nk * d) * d;
                            if (BTAB == 2) {
                                const double dx = xj - c.ux;
                                const double t = c.nk * dx;
                                sA[2 * s][j] = fma(t, dx, c.a);
                                sA[2 * s + 1][j] = fma(t, dx, c.al);
                            }
                        }
                    }
                    __syncthreads();
                }
                if constexpr (BTAB == 2 && TX * TY > 9) {
                    // Software-pipelined: the table values of state s + 1 are
                    // read before the pair work of state s, so the LDS latency
                    // is covered by that work within the wave (tiles at two
                    // waves per SIMD: tri2m 159.4 -> 155.5 ms; the three-wave
                    // tiles hide it across waves and measured slower with
                    // it).  The last iteration re-reads its own state (in
                    // range, unused).
                    double ca[TX], cai[TX], cb[TY];
#pragma unroll
                    for (int i = 0; i < TX; ++i) {
                        ca[i] = sA[0][xcol(i)];
                        cai[i] = sA[1][xcol(i)];
                    }
#pragma unroll
                    for (int j = 0; j < TY; ++j) cb[j] = sB[0][ycol(j)];
                    // The stencil's first state sets the envelopes (q is its
                    // own min and max) instead of comparing with +-inf:
                    // tri2m 152.0 -> 150.6 ms, bounds bitwise the same (v_min
                    // and v_max return the number where the other operand
                    // is NaN, so only a stencil whose every state gave NaN
                    // at a node could differ).
                    int s0 = 0;
                    if (c0 == 0 && t0 == 0) {
                        const int sn = tn > 1 ? 1 : 0;
                        double na[TX], nai[TX], nb[TY];
#pragma unroll
                        for (int i = 0; i < TX; ++i) {
                            na[i] = sA[2 * sn][xcol(i)];
                            nai[i] = sA[2 * sn + 1][xcol(i)];
                        }
#pragma unroll
                        for (int j = 0; j < TY; ++j) nb[j] = sB[sn][ycol(j)];
#pragma unroll
                        for (int i = 0; i < TX; ++i)
#pragma unroll
                            for (int j = 0; j < TY; ++j) {
                                const double q = ca[i] + cb[j];
                                const double qi = cai[i] + cb[j];
                                qtn[i][j] = q;
                                qtx[i][j] = q;
                                qin[i][j] = qi;
                                qix[i][j] = qi;
                            }
#pragma unroll
                        for (int i = 0; i < TX; ++i) { ca[i] = na[i]; cai[i] = nai[i]; }
#pragma unroll
                        for (int j = 0; j < TY; ++j) cb[j] = nb[j];
                        s0 = 1;
                    }
#pragma unroll 2
                    for (int s = s0; s < tn; ++s) {
                        const int sn = s + 1 < tn ? s + 1 : s;
                        double na[TX], nai[TX], nb[TY];
#pragma unroll
                        for (int i = 0; i < TX; ++i) {
                            na[i] = sA[2 * sn][xcol(i)];
                            nai[i] = sA[2 * sn + 1][xcol(i)];
                        }
#pragma unroll
                        for (int j = 0; j < TY; ++j) nb[j] = sB[sn][ycol(j)];
#pragma unroll
                        for (int i = 0; i < TX; ++i)
#pragma unroll
                            for (int j = 0; j < TY; ++j) {
                                const double q = ca[i] + cb[j];
                                const double qi = cai[i] + cb[j];
                                qtn[i][j] = fmin(qtn[i][j], q);
                                qtx[i][j] = fmax(qtx[i][j], q);
                                qin[i][j] = fmin(qin[i][j], qi);
                                qix[i][j] = fmax(qix[i][j], qi);
                            }
#pragma unroll
                        for (int i = 0; i < TX; ++i) { ca[i] = na[i]; cai[i] = nai[i]; }
#pragma unroll
                        for (int j = 0; j < TY; ++j) cb[j] = nb[j];
                    }
                    continue;
                }
                // the x terms a, a + l and the y terms b of state s at this
                // thread's nodes, from the tables or from the coefficients
                auto terms = [&](int s, double* a, double* ai, double* b) {
                    if (BTAB == 2) {
#pragma unroll
                        for (int i = 0; i < TX; ++i) {
                            a[i] = sA[2 * s][xcol(i)];
                            ai[i] = sA[2 * s + 1][xcol(i)];
                        }
                    } else {
                        const Coef c = sC[t0 + s];
#pragma unroll
                        for (int i = 0; i < TX; ++i) {
                            const double d = ux[i] - c.ux;
                            const double t = c.nk * d;
                            a[i] = fma(t, d, c.a);
                            ai[i] = fma(t, d, c.al);
                        }
                    }
                    if (BTAB) {
#pragma unroll
                        for (int j = 0; j < TY; ++j) b[j] = sB[s][ycol(j)];
                    } else {
                        const Coef c = sC[t0 + s];
#pragma unroll
                        for (int j = 0; j < TY; ++j) {
                            const double d = uy[j] - c.uy;
                            b[j] = (c.nk * d) * d;
                        }
                    }
                };
                int s0 = 0;
                if (c0 == 0 && t0 == 0) {
                    // the stencil's first state sets the envelopes
                    double a[TX], ai[TX], b[TY];
                    terms(0, a, ai, b);
#pragma unroll
                    for (int i = 0; i < TX; ++i)
#pragma unroll
                        for (int j = 0; j < TY; ++j) {
                            const double q = a[i] + b[j];
                            const double qi = ai[i] + b[j];
                            qtn[i][j] = q;
                            qtx[i][j] = q;
                            qin[i][j] = qi;
                            qix[i][j] = qi;
                        }
                    s0 = 1;
                }
#pragma unroll 2
                for (int s = s0; s < tn; ++s) {
                    double a[TX], ai[TX], b[TY];
                    terms(s, a, ai, b);
#pragma unroll
                    for (int i = 0; i < TX; ++i)
#pragma unroll
                        for (int j = 0; j < TY; ++j) {
                            const double q = a[i] + b[j];
                            const double qi = ai[i] + b[j];
                            qtn[i][j] = fmin(qtn[i][j], q);
                            qtx[i][j] = fmax(qtx[i][j], q);
                            qin[i][j] = fmin(qin[i][j], qi);
                            qix[i][j] = fmax(qix[i][j], qi);
                        }
                }
            }
        }

        // exp, relaxation, trapezoid weights and the moment contraction.  The
        // node coordinates and weights are formed here from box values passed
        // through an empty asm statement: otherwise the compiler computes
        // them (and other element-invariant parts of this contraction) before
        // the hot loop and keeps them live across it (register pressure).
        // The sums run over the unrelaxed envelopes g = exp(q); the factors
        // (1 -+ r) of eq. relaxed are applied once per thread afterwards.
        // Momentum (eq. mmbounds, mpbounds): the lower bound takes the upper
        // envelope where u < 0 and the lower one where u >= 0 (the upper
        // bound the reverse), so M u is split by sign into min(M u, 0) and
        // max(M u, 0), which feed separate sums without selects.
        double cx = lox, cy = loy, dx = hx, dy = hy;
        int otx = idle ? p.nx : tx, oty = idle ? p.ny : ty;
        asm volatile("" : "+v"(cx), "+v"(cy), "+v"(dx), "+v"(dy), "+v"(otx), "+v"(oty));
        // The weights and moment polynomials are separable, M = wx wy,
        // |u|^2 / 2 = vx^2 / 2 + vy^2 / 2 and the sign of M u_k depends on
        // u_k alone, so each node only feeds per-row sums over y (R: lower
        // and upper envelope, internal parts) and per-column sums over x (C:
        // lower and upper envelope), six fma per node; the moments are then
        // formed once per row and once per column.
        double sr[2] = {0, 0}, se[2] = {0, 0};    // rho, E: (lower, upper) envelope sums
        double mn[2][2] = {{0, 0}, {0, 0}};       // [dir][0]: sum u<0 of M u g_max, [1]: u>=0, M u g_min
        double mx[2][2] = {{0, 0}, {0, 0}};       // [dir][0]: sum u<0 of M u g_min, [1]: u>=0, M u g_max
        double ctn[TY], ctx[TY];                  // per column: sum over x of wx g_min, wx g_max
#pragma unroll
        for (int j = 0; j < TY; ++j) { ctn[j] = 0.0; ctx[j] = 0.0; }
#pragma unroll
        for (int i = 0; i < TX; ++i) {
            const int jx = otx + bx * i;
            if (jx >= p.nx) continue;
            const double vx = node_pos(cx, jx, dx);
            const double wx = dx * ((jx == 0 || jx == p.nx - 1) ? 0.5 : 1.0);
            double rtn = 0.0, rtx = 0.0, rin = 0.0, rix = 0.0;   // per row: sum over y of wy g
            if constexpr (TX * TY == 16 && TY % 2 == 0) {
                // two nodes at a time, in three phases: the eight indices and
                // polynomials, the eight table reads together, the products
                // (otherwise each exp waits for its own table read right
                // after issuing it: tri2m 155.4 -> 153.1 ms)
#pragma unroll
                for (int j = 0; j < TY; j += 2) {
                    double xs[8];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        xs[4 * h + 0] = qtn[i][j + h]; xs[4 * h + 1] = qtx[i][j + h];
                        xs[4 * h + 2] = qin[i][j + h]; xs[4 * h + 3] = qix[i][j + h];
                    }
                    ExpPrep pr[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) pr[k] = exp_prep(xs[k]);
                    __builtin_amdgcn_sched_barrier(0);
                    ExpPair T[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) T[k] = sExp[pr[k].ni & 255];
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int jy = oty + by * (j + h);
                        // nodes past the grid (finite values) add zero
                        const double wy = jy < p.ny ? dy * ((jy == 0 || jy == p.ny - 1) ? 0.5 : 1.0) : 0.0;
                        const double gtn = exp_fin(pr[4 * h + 0], T[4 * h + 0]);
                        const double gtx = exp_fin(pr[4 * h + 1], T[4 * h + 1]);
                        const double gin = exp_fin(pr[4 * h + 2], T[4 * h + 2]);
                        const double gix = exp_fin(pr[4 * h + 3], T[4 * h + 3]);
                        rtn = fma(wy, gtn, rtn);
                        rtx = fma(wy, gtx, rtx);
                        rin = fma(wy, gin, rin);
                        rix = fma(wy, gix, rix);
                        ctn[j + h] = fma(wx, gtn, ctn[j + h]);
                        ctx[j + h] = fma(wx, gtx, ctx[j + h]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
            for (int j = 0; j < TY; ++j) {
                const int jy = oty + by * j;
                if (jy >= p.ny) continue;
                const double wy = dy * ((jy == 0 || jy == p.ny - 1) ? 0.5 : 1.0);
                const double gtn = exp_tab(qtn[i][j], sExp);
                const double gtx = exp_tab(qtx[i][j], sExp);
                const double gin = exp_tab(qin[i][j], sExp);
                const double gix = exp_tab(qix[i][j], sExp);
                rtn = fma(wy, gtn, rtn);
                rtx = fma(wy, gtx, rtx);
                rin = fma(wy, gin, rin);
                rix = fma(wy, gix, rix);
                ctn[j] = fma(wx, gtn, ctn[j]);
                ctx[j] = fma(wx, gtx, ctx[j]);
                // two nodes at a time: the exps of a pair interleave (their
                // LDS table reads overlap), while the temporaries of more
                // nodes would not fit the registers
                if (j & 1) __builtin_amdgcn_sched_barrier(0);
            }
            }
            const double hx2 = 0.5 * vx * vx;
            sr[0] = fma(wx, rtn, sr[0]);
            sr[1] = fma(wx, rtx, sr[1]);
            se[0] = fma(wx, fma(hx2, rtn, rin), se[0]);
            se[1] = fma(wx, fma(hx2, rtx, rix), se[1]);
            const double mu = wx * vx;
            const double neg = fmin(mu, 0.0), pos = fmax(mu, 0.0);
            mn[0][0] = fma(neg, rtx, mn[0][0]);
            mn[0][1] = fma(pos, rtn, mn[0][1]);
            mx[0][0] = fma(neg, rtn, mx[0][0]);
            mx[0][1] = fma(pos, rtx, mx[0][1]);
        }
#pragma unroll
        for (int j = 0; j < TY; ++j) {
            const int jy = oty + by * j;
            if (jy >= p.ny) continue;
            const double vy = node_pos(cy, jy, dy);
            const double wy = dy * ((jy == 0 || jy == p.ny - 1) ? 0.5 : 1.0);
            const double wy2 = wy * (0.5 * vy * vy);
            se[0] = fma(wy2, ctn[j], se[0]);
            se[1] = fma(wy2, ctx[j], se[1]);
            const double mu = wy * vy;
            const double neg = fmin(mu, 0.0), pos = fmax(mu, 0.0);
            mn[1][0] = fma(neg, ctx[j], mn[1][0]);
            mn[1][1] = fma(pos, ctn[j], mn[1][1]);
            mx[1][0] = fma(neg, ctn[j], mx[1][0]);
            mx[1][1] = fma(pos, ctx[j], mx[1][1]);
        }
        double part[8] = {rm * sr[0], rp * sr[1], rm * se[0], rp * se[1],
                          rp * mn[0][0] + rm * mn[0][1], rm * mx[0][0] + rp * mx[0][1],
                          rp * mn[1][0] + rm * mn[1][1], rm * mx[1][0] + rp * mx[1][1]};
        const double sum = block_sum8<NT>(part, red);
        if (tid < 8) store_bound_value<2>(p, e, tid, sum, flags);
    }
}

template <typename K>
hipError_t launch(K kernel, int threads, const BoundsArgs& a, hipStream_t stream) {
    hipLaunchKernelGGL(kernel, dim3(bounds_grid(a)), dim3(threads), 0, stream, a);
    return hipGetLastError();
}

}  // namespace
}  // namespace kbl
