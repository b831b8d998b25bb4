// Shared by the translation units of the 1D flux reconstruction solver: the
// inviscid fluxes and the arguments of a limited stage.
#pragma once

#include "../../include/kbl_fr1d.h"
#include "kbl_internal.h"

namespace kbl {

constexpr int kFrNs = KBL_FR_MAX_DEGREE + 1;

// Arguments of one limited stage, by value.  Operators padded with zeros to
// kFrNs nodes.
struct FrStageArgs {
    const double* A;      // stage input [3][a_stride]
    const double* U0;     // state at the start of the step [3][u0_stride]
    double* B;            // stage output [3][b_stride]; not A
    uint32_t* status;     // [n_launch] limiter status or null
    int64_t a_stride, u0_stride, b_stride;
    int64_t n_elem;
    int64_t n_launch;     // elements to write: n_elem, or with the ghosts
    int32_t n_s, n_v;     // solution points, nodes (p + 1, p + 3)
    int32_t bc;
    int32_t first;        // the input's end values are not current
    double inv_jac;       // 2 / h
    double lhd;           // ln(delta / (4 pi)); unused without internal degrees of freedom
    double gamma, gm1;
    double left[3], right[3];
    double ca, cb, dt;    // out <- ca U0 + cb (A + dt R(A)), limited
    const double* tdt;    // device (t, dt): dt read from tdt[1] when not null
    double at[2][kFrNs];  // l_j(-1), l_j(+1)
    double D[kFrNs][kFrNs];   // l_k'(x_j)
    double dg[2][kFrNs];  // g_L'(x_j), g_R'(x_j)
    BoundsArgs b;
    LimitArgs l;
};

hipError_t launch_fr1d_stage_limited(const FrStageArgs& f, hipStream_t stream);

__device__ __forceinline__ void fr_euler_flux(double gm1, const double w[3], double f[3]) {
#pragma clang fp contract(off)
    const double u = w[1] / w[0];
    const double P = gm1 * (w[2] - 0.5 * w[1] * u);
    f[0] = w[1];
    f[1] = w[1] * u + P;
    f[2] = (w[2] + P) * u;
}

// HLLC flux (Toro, Spruce and Speares) with the speeds
// S_L = min(u_L - c_L, u_R - c_R), S_R = max(u_L + c_L, u_R + c_R).
__device__ __forceinline__ void fr_hllc(double gamma, double gm1, const double L[3],
                                        const double Rr[3], double F[3]) {
#pragma clang fp contract(off)
    const double ul = L[1] / L[0], ur = Rr[1] / Rr[0];
    const double pl = gm1 * (L[2] - 0.5 * L[1] * ul);
    const double pr = gm1 * (Rr[2] - 0.5 * Rr[1] * ur);
    const double cl = sqrt(gamma * pl / L[0]), cr = sqrt(gamma * pr / Rr[0]);
    const double SL = fmin(ul - cl, ur - cr);
    const double SR = fmax(ul + cl, ur + cr);
    const double dl = L[0] * (SL - ul), dr = Rr[0] * (SR - ur);
    const double Ss = (pr - pl + ul * dl - ur * dr) / (dl - dr);
    double fl[3], fr[3];
    fr_euler_flux(gm1, L, fl);
    fr_euler_flux(gm1, Rr, fr);
    if (0.0 <= SL) {
        F[0] = fl[0]; F[1] = fl[1]; F[2] = fl[2];
    } else if (0.0 <= Ss) {
        const double k = dl / (SL - Ss);
        const double e = k * (L[2] / L[0] + (Ss - ul) * (Ss + pl / dl));
        F[0] = fl[0] + SL * (k - L[0]);
        F[1] = fl[1] + SL * (k * Ss - L[1]);
        F[2] = fl[2] + SL * (e - L[2]);
    } else if (0.0 <= SR) {
        const double k = dr / (SR - Ss);
        const double e = k * (Rr[2] / Rr[0] + (Ss - ur) * (Ss + pr / dr));
        F[0] = fr[0] + SR * (k - Rr[0]);
        F[1] = fr[1] + SR * (k * Ss - Rr[1]);
        F[2] = fr[2] + SR * (e - Rr[2]);
    } else {
        F[0] = fr[0]; F[1] = fr[1]; F[2] = fr[2];
    }
}

}  // namespace kbl
