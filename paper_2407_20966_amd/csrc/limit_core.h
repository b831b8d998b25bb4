// The squeeze limiter and pressure step of one element held by an aligned
// group of lanes (Sec. 3.4, Sec. 3.8), shared by the limiter kernel and the
// fused stage of the 1D solver.
#pragma once

#include <math.h>

#include "kbl_internal.h"

namespace kbl {
namespace limiter {

constexpr double kInf = __builtin_inf();

// Group exchanges.  Stage k pairs each lane with a partner in the other
// half of its aligned block of 2^(k+1) lanes: inside a row of 16 on the DPP
// network (quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror,
// row_mirror), across rows (groups of 32 or 64 lanes) by shuffles.  After
// the last stage every lane of the group holds the same combination.
constexpr int kDppQuadXor1 = 0xB1;
constexpr int kDppQuadXor2 = 0x4E;
constexpr int kDppRowHalfMirror = 0x141;
constexpr int kDppRowMirror = 0x140;

template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = dpp_i32<CTRL>((int)b);
    const int hi = dpp_i32<CTRL>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
// The partner of stage `o` (block half-size o = 1, 2, 4, ... G/2).
template <int O>
__device__ __forceinline__ double grp_partner(double v) {
    if (O == 1) return dpp_f64<kDppQuadXor1>(v);
    if (O == 2) return dpp_f64<kDppQuadXor2>(v);
    if (O == 4) return dpp_f64<kDppRowHalfMirror>(v);
    if (O == 8) return dpp_f64<kDppRowMirror>(v);
    return __shfl_xor(v, O, 64);
}
template <int O>
__device__ __forceinline__ int grp_partner_i32(int v) {
    if (O == 1) return dpp_i32<kDppQuadXor1>(v);
    if (O == 2) return dpp_i32<kDppQuadXor2>(v);
    if (O == 4) return dpp_i32<kDppRowHalfMirror>(v);
    if (O == 8) return dpp_i32<kDppRowMirror>(v);
    return __shfl_xor(v, O, 64);
}
template <int G, class F>
__device__ __forceinline__ double grp_reduce(double v, F f) {
    if (G >= 2) v = f(v, grp_partner<1>(v));
    if (G >= 4) v = f(v, grp_partner<2>(v));
    if (G >= 8) v = f(v, grp_partner<4>(v));
    if (G >= 16) v = f(v, grp_partner<8>(v));
    if (G >= 32) v = f(v, grp_partner<16>(v));
    if (G >= 64) v = f(v, grp_partner<32>(v));
    return v;
}
template <int G>
__device__ __forceinline__ double grp_sum(double v) {
    return grp_reduce<G>(v, [](double a, double b) { return a + b; });
}
template <int G>
__device__ __forceinline__ double grp_min(double v) {
    return grp_reduce<G>(v, [](double a, double b) { return fmin(a, b); });
}
template <int G>
__device__ __forceinline__ double grp_max(double v) {
    return grp_reduce<G>(v, [](double a, double b) { return fmax(a, b); });
}

template <int D>
__device__ __forceinline__ double pressure(double gm1, const double* w) {
    double mm = w[1] * w[1];
#pragma unroll
    for (int j = 2; j <= D; ++j) mm += w[j] * w[j];
    return gm1 * (w[D + 1] - 0.5 * mm / w[0]);
}

// Limits one element.  Lane j of the group holds node j: w (live: j < n_s),
// its mean weight c (0 if not live) and the element's bounds b; bad_b: some
// bound is not finite, the element passes through.  Out: the limited node wt,
// alpha_min, alpha_P and the status, the last three the same in every lane of
// the group.  All lanes of the wave take part.
template <int D, int G>
__device__ __forceinline__ void limit_group(const LimitArgs& p, const double (&w)[D + 2],
                                            const double (&b)[2 * (D + 2)], double c, bool live,
                                            bool bad_b, double (&wt)[D + 2], double& amin,
                                            double& aP, uint32_t& st) {
    constexpr int NV = D + 2;
    // alpha_v = min(1, |b_max - wbar| / |w_max - wbar|, |b_min - wbar| /
    // |w_min - wbar|) (eq. alpha).  The ratios are ordered by cross products
    // of their (non-negative) numerators and denominators, which are bounded
    // below by eps, and only the smallest is divided: one division per
    // element for the coupled minimum, one per component when independent.
    st = 0;
    double wbar[NV], rn[NV], rd[NV];
    bool eps0 = false;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        wbar[v] = grp_sum<G>(c * w[v]) * p.inv_csum;
        const double wmax = grp_max<G>(live ? w[v] : -kInf);
        const double wmin = grp_min<G>(live ? w[v] : kInf);
        if (wbar[v] < b[v] || wbar[v] > b[NV + v]) st |= KBL_ST_MEAN_OUTSIDE;
        const double du = fabs(wmax - wbar[v]), dl = fabs(wmin - wbar[v]);
        const double nu = fabs(b[NV + v] - wbar[v]), nl = fabs(b[v] - wbar[v]);
        const bool lo = nl * du < nu * dl;          // the lower side binds first
        const bool ev = dl < p.eps || du < p.eps;
        eps0 |= ev;
        rn[v] = ev ? 0.0 : (lo ? nl : nu);          // ratio 0 under the eps rule
        rd[v] = ev ? 1.0 : (lo ? dl : du);
    }
    if (eps0) st |= KBL_ST_EPS_RULE;
    double acomp[NV];
    if (!p.independent) {
        double Nm = 1.0, Dm = 1.0;                  // smallest ratio, as Nm / Dm
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (rn[v] * Dm < Nm * rd[v]) { Nm = rn[v]; Dm = rd[v]; }
        amin = Nm < Dm ? Nm / Dm : 1.0;
#pragma unroll
        for (int v = 0; v < NV; ++v) acomp[v] = amin;
    } else {
        amin = 1.0;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            acomp[v] = rn[v] < rd[v] ? rn[v] / rd[v] : 1.0;
            amin = fmin(amin, acomp[v]);
        }
    }
    if (amin < 1.0) st |= KBL_ST_LIMITED;

    // coupled (eq. limiter) or independent per-component blend
#pragma unroll
    for (int v = 0; v < NV; ++v) wt[v] = wbar[v] + acomp[v] * (w[v] - wbar[v]);

    double P = live ? pressure<D>(p.gm1, wt) : kInf;
    if (isnan(P)) P = -kInf;
    const double pmin = grp_min<G>(P);
    aP = 1.0;
    if (pmin < p.p_floor) {
        st |= KBL_ST_PSTEP;
        const double pbar = pressure<D>(p.gm1, wbar);
        if (pbar > p.p_floor) aP = fabs((p.p_floor - pbar) / (pmin - pbar));
        else { aP = 0.0; st |= KBL_ST_PMEAN_FLOOR; }
#pragma unroll
        for (int v = 0; v < NV; ++v) wt[v] = wbar[v] + aP * (wt[v] - wbar[v]);
    }

    if (bad_b) {
        st = KBL_ST_BAD_BOUNDS;
        amin = 1.0;
        aP = 1.0;
#pragma unroll
        for (int v = 0; v < NV; ++v) wt[v] = w[v];
    }
}

}  // namespace limiter
}  // namespace kbl
