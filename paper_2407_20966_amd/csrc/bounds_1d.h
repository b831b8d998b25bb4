// One-dimensional velocity grids: envelopes of a few nodes per thread and their
// moments, shared by the 1D bounds kernel and the fused stage of the 1D solver.
#pragma once

#include "bounds_common.h"

namespace kbl {
namespace {

// min and max of values known to be numbers (one instruction also where the
// translation unit honours NaNs and would canonicalise the operands first).
__device__ __forceinline__ double raw_min(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double raw_max(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// exp_prep's clamp likewise.
__device__ __forceinline__ ExpPrep raw_exp_prep(double x) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(x), "s"(-1100.0));
    return exp_prep_clamped(r);
}

// Unrelaxed envelope sums of a 1D velocity grid: rho, E (lower, upper) and the
// momentum split by the sign of u.
struct Sums1D {
    double sr[2] = {0, 0}, se[2] = {0, 0}, mn[2] = {0, 0}, mx[2] = {0, 0};
    // the six relaxed sums in the order of store_bounds
    __device__ __forceinline__ void parts(double rm, double rp, double* part) const {
        part[0] = rm * sr[0];
        part[1] = rp * sr[1];
        part[2] = rm * se[0];
        part[3] = rp * se[1];
        part[4] = rp * mn[0] + rm * mn[1];
        part[5] = rm * mx[0] + rp * mx[1];
        part[6] = part[7] = 0.0;
    }
};

// Envelopes of T nodes of a 1D velocity grid (node j0 + stride i) and their
// moments.  No separability to exploit: a pair costs sub, mul and two fma
// before the four min/max.  Coefficients are broadcast from LDS.
template <int T>
struct Env1D {
    double qtn[T], qtx[T], qin[T], qix[T];
    __device__ __forceinline__ static double node(const BoundsArgs& p, double lo, double h, int j) {
        return node_pos(lo, j < p.nx ? j : p.nx - 1, h);
    }
    // States [0, cn) of sC; first: they set the envelopes (no +-inf starting
    // values) instead of being compared with them.
    __device__ __forceinline__ void fold(const BoundsArgs& p, const Coef* sC, int cn, double lo,
                                         double h, int j0, int stride, bool first) {
        double u[T];
#pragma unroll
        for (int i = 0; i < T; ++i) u[i] = node(p, lo, h, j0 + stride * i);
        int s = 0;
        if (first) {
            const Coef c = sC[0];
#pragma unroll
            for (int i = 0; i < T; ++i) {
                const double d = u[i] - c.ux;
                const double t = c.nk * d;
                qtn[i] = qtx[i] = fma(t, d, c.a);
                qin[i] = qix[i] = fma(t, d, c.al);
            }
            s = 1;
        }
        for (; s < cn; ++s) {
            const Coef c = sC[s];
#pragma unroll
            for (int i = 0; i < T; ++i) {
                const double d = u[i] - c.ux;
                const double t = c.nk * d;
                const double q = fma(t, d, c.a);
                const double qi = fma(t, d, c.al);
                qtn[i] = raw_min(qtn[i], q);
                qtx[i] = raw_max(qtx[i], q);
                qin[i] = raw_min(qin[i], qi);
                qix[i] = raw_max(qix[i], qi);
            }
        }
    }
    // Adds the nodes' moments to the unrelaxed envelope sums (the momentum
    // sums split M u by sign, as in the 2D kernel).
    __device__ __forceinline__ void contract(const BoundsArgs& p, double lo, double h, int j0,
                                             int stride, const ExpPair* tab, Sums1D& m) const {
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int j = j0 + stride * i;
            // the four exps in three phases: indices and polynomials, the
            // table reads together, the products
            const ExpPrep p0 = raw_exp_prep(qtn[i]), p1 = raw_exp_prep(qtx[i]);
            const ExpPrep p2 = raw_exp_prep(qin[i]), p3 = raw_exp_prep(qix[i]);
            const ExpPair t0 = tab[p0.ni & 255], t1 = tab[p1.ni & 255];
            const ExpPair t2 = tab[p2.ni & 255], t3 = tab[p3.ni & 255];
            const double u = node(p, lo, h, j);
            // nodes past the grid (finite values) add zero
            const double M = j < p.nx ? h * ((j == 0 || j == p.nx - 1) ? 0.5 : 1.0) : 0.0;
            const double gtn = exp_fin(p0, t0), gtx = exp_fin(p1, t1);
            const double gin = exp_fin(p2, t2), gix = exp_fin(p3, t3);
            const double hu2 = 0.5 * u * u;
            m.sr[0] += M * gtn;
            m.sr[1] += M * gtx;
            m.se[0] += M * (hu2 * gtn + gin);
            m.se[1] += M * (hu2 * gtx + gix);
            const double mu = M * u;
            const double neg = fmin(mu, 0.0), pos = fmax(mu, 0.0);
            m.mn[0] += neg * gtx;
            m.mn[1] += pos * gtn;
            m.mx[0] += neg * gtn;
            m.mx[1] += pos * gtx;
            __builtin_amdgcn_sched_barrier(0);
        }
    }
};

}  // namespace
}  // namespace kbl
