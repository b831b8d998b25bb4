// One-dimensional velocity grids: envelopes of a few nodes per thread and their
// moments, shared by the 1D bounds kernel and the fused stage of the 1D solver.
#pragma once

#include <type_traits>

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

// Which of S <= 64 staged states can hold an extremum of g or g_I at the wave's
// nodes of a round: the wave owns 64 T consecutive nodes of a round of NT T.
// With c the middle of those nodes, w their half width and r the state whose q
// is largest at c,
//   q_i - q_r <= (q_i - q_r)(c) + w |dg| + w^2 max(nk_i - nk_r, 0),
// and a state for which that plus max(l_i - l_r, 0) is negative is neither
// maximum; likewise from below.  Half widths are widened by 1e-10 and thresholds by
// 1e-12, far above rounding, so the envelopes are those of all states.
// 64 / 2^lg rounds from `round` on at once: lane = (round, state mod 2^lg).
// Returns their masks side by side; the mask of a round past the grid is 0.
template <int NT, int T>
__device__ __forceinline__ unsigned long long cull_1d(const BoundsArgs& p, const Coef* sC, int S,
                                                      double lo, double h, int round, int lg) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int s = lane & ((1 << lg) - 1);
    const int ja = (round + (lane >> lg)) * NT * T + wid * 64 * T;
    const int jb = min(ja + 64 * T, p.nx) - 1;
    const double x0 = node_pos(lo, ja, h), x1 = node_pos(lo, jb, h);
    const double cx = 0.5 * (x0 + x1);
    // twice the half width (the gradients below are halved), widened
    const double w = fabs(x1 - x0) * (1.0 + 1e-10) + 1e-14 * (fabs(x0) + fabs(x1));
    const double Q = 0.25 * w * w;
    const bool internal = p.half_delta > 0.0, live = s < S;
    const Coef c = sC[live ? s : 0];
    const double d = cx - c.ux, t = c.nk * d, v = fma(t, d, c.a), qn = Q * c.nk;
    const double l = internal ? c.al - c.a : 0.0;
    // q less the first state's, the state's index in the low bits: the reference
    // found is the extremum up to 2^-17 of the states' spread, however little they
    // differ, and any state is a valid reference
    const Coef& f = sC[0];
    const double d0 = cx - f.ux, v0 = fma(f.nk * d0, d0, f.a);
    const float key = __int_as_float((__float_as_int((float)(v - v0)) & ~63) | s);
    float kmax = live ? key : -kInfF, kmin = live ? key : kInfF;
    auto dpp = [](float x, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x),
                                                          decltype(ctrl)::value, 0xF, 0xF, false));
    };
    auto step = [&](auto ctrl) {
        kmax = fmaxf(kmax, dpp(kmax, ctrl));
        kmin = fminf(kmin, dpp(kmin, ctrl));
    };
    step(std::integral_constant<int, kDppXor1>{});
    step(std::integral_constant<int, kDppXor2>{});
    step(std::integral_constant<int, kDppHalfMirror>{});
    step(std::integral_constant<int, kDppMirror>{});
    for (int o = 16; o < (1 << lg); o <<= 1) {
        kmax = fmaxf(kmax, __shfl_xor(kmax, o, 64));
        kmin = fminf(kmin, __shfl_xor(kmin, o, 64));
    }
    unsigned long long keep = 0;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const Coef r = sC[__float_as_int(side ? kmin : kmax) & 63];
        const double dr = cx - r.ux, tr = r.nk * dr, vr = fma(tr, dr, r.a), qr = Q * r.nk;
        const double lr = internal ? r.al - r.a : 0.0;
        const double slack = 1e-12 * (1.0 + fabs(vr) + fabs(r.a) + w * fabs(tr) + fabs(qr) + fabs(lr));
        const double sg = side ? -1.0 : 1.0;
        const double b = fma(w, fabs(t - tr), sg * (v - vr)) + fmax(sg * (l - lr), 0.0) +
                         fmax(sg * (qn - qr), 0.0);
        constexpr int kNotBelow = 11;    // also where no bound is finite (a denormal temperature)
        keep |= __builtin_amdgcn_fcmp(b, -slack, kNotBelow);
    }
    const unsigned long long in_grid = __builtin_amdgcn_ballot_w64(live && ja < p.nx);
    keep &= in_grid;
    if (keep == in_grid) {
        // every state is kept: where all are the same (a constant field) the first
        // stands for them
        if (__builtin_amdgcn_ballot_w64(c.a != f.a || c.al != f.al || c.ux != f.ux || c.nk != f.nk) == 0)
            keep &= __builtin_amdgcn_ballot_w64(s == 0);
    }
    return keep;
}

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
    // The states of a mask (not 0, the same in every lane); the next state's
    // coefficients are read before the current state's work.
    __device__ __forceinline__ void fold_mask(const BoundsArgs& p, const Coef* sC,
                                              unsigned long long m, double lo, double h, int j0,
                                              int stride) {
        double u[T];
#pragma unroll
        for (int i = 0; i < T; ++i) u[i] = node(p, lo, h, j0 + stride * i);
        auto next = [&]() {
            const int s = __builtin_ctzll(m);
            m &= m - 1;
            return sC[s];
        };
        Coef c = next();
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const double d = u[i] - c.ux;
            const double t = c.nk * d;
            qtn[i] = qtx[i] = fma(t, d, c.a);
            qin[i] = qix[i] = fma(t, d, c.al);
        }
        if (m == 0) return;
        Coef n = next();
        for (;;) {
            c = n;
            const bool last = m == 0;
            if (!last) n = next();
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
            if (last) break;
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
