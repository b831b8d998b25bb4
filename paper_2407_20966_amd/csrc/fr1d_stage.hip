// One limited SSP-RK stage of the 1D flux reconstruction solver in one kernel
// (the overview of Sec. 3.9): bounds of the stage's input state over the node
// stencils, the update, and the limiting of the updated element into those
// bounds, gfx950.
//
// One workgroup owns one element.  The stage reads its input from one buffer
// and writes another, so that an element's workgroup may read its neighbours
// at any time.  The small steps go to different waves, which run them at the
// same time:
//  - wave 0: the log-Maxwellians of the p + 5 stencil states and the velocity
//    box, lane = state;
//  - wave 1: the FR residual and the stage update, lanes = nodes;
//  - all waves: the envelopes and moments over the velocity nodes, as in
//    bounds_fp64_1d;
//  - wave 2: the limiter and the store.
// The stencil is the mesh's own (element and face neighbours), so no index
// arrays are read, and the bounds, the residual and the unlimited state never
// leave the workgroup.  p enters as a loop bound only: the operators are
// padded with zeros to eight nodes.
//
// What bounds it: VALU issue, 141 ops per velocity node (p = 3) and about 1900
// per element for the small steps.  A step of 3200 elements on 2048 velocity
// nodes takes 132 us in three launches, against 204 in fourteen with separate
// kernels for the end values, the bounds (150 us of it), the residual, the
// update and the limiter; 12000 elements 417 against 531 us; 50 elements on
// 512 nodes, all latency, 26 against 66 us.  Two velocity nodes per thread and
// round leave 82 VGPRs, six waves per SIMD: four nodes in 102 VGPRs take 140 us,
// 128 or 64 threads per element 136 and 150, a cap of 72 VGPRs (seven waves,
// 14 spills) 137.
#include "bounds_1d.h"
#include "fr1d_internal.h"
#include "limit_core.h"

namespace kbl {
namespace {

// The wave's own LDS accesses execute in program order; this only keeps the
// compiler from moving accesses of other lanes' data across it.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Where an element's node values come from: its columns of the stage input,
// or a constant state (the ghosts of Dirichlet boundaries).
struct FrElem {
    int64_t col;
    int ghost;   // 0: element; 1: left, 2: right constant state
};
__device__ __forceinline__ FrElem fr_elem(const FrStageArgs& f, int64_t e) {
    FrElem r{e * f.n_v, 0};
    if (f.bc == KBL_FR_PERIODIC) {
        if (e < 0) r.col = (f.n_elem - 1) * f.n_v;
        if (e >= f.n_elem) r.col = 0;
    } else if (e < 0 || e >= f.n_elem) {
        r.col = 0;
        r.ghost = e < 0 ? 1 : 2;
    }
    return r;
}
__device__ __forceinline__ double fr_const(const FrStageArgs& f, const FrElem& r, int v) {
    return r.ghost == 1 ? f.left[v] : f.right[v];
}

// Lagrange interpolation of an element's solution points to one end (0: x = -1,
// 1: x = +1); the same operations in the same order wherever it is used.
__device__ __forceinline__ double fr_end_dot(const FrStageArgs& f, int end,
                                             const double (&u)[kFrNs]) {
    double s = (end ? f.at[1][0] : f.at[0][0]) * u[0];
#pragma unroll
    for (int j = 1; j < kFrNs; ++j) s = fma(end ? f.at[1][j] : f.at[0][j], u[j], s);
    return s;
}
__device__ __forceinline__ void fr_ends(const FrStageArgs& f, const FrElem& r, int end,
                                        double (&w)[3]) {
    double u[3][kFrNs];
#pragma unroll
    for (int v = 0; v < 3; ++v)
#pragma unroll
        for (int j = 0; j < kFrNs; ++j)
            u[v][j] = f.A[v * f.a_stride + r.col + (j < f.n_s ? j : 0)];
#pragma unroll
    for (int v = 0; v < 3; ++v) {
#pragma unroll
        for (int j = 0; j < kFrNs; ++j) u[v][j] = j < f.n_s ? u[v][j] : 0.0;
        w[v] = fr_end_dot(f, end, u[v]);
    }
}

// Stencil state s of element e (Sec. 5): its solution points and end values,
// then the left neighbour's right end and the right neighbour's left end.  In
// the first stage the end values are the interpolants of the solution points.
__device__ __forceinline__ void stencil_state(const FrStageArgs& f, int64_t e, int s,
                                              double (&w)[3]) {
    const int64_t en = e + (s == f.n_v ? -1 : s == f.n_v + 1 ? 1 : 0);
    const int idx = s == f.n_v ? f.n_s + 1 : s == f.n_v + 1 ? f.n_s : s;
    const FrElem r = fr_elem(f, en);
    if (r.ghost) {
#pragma unroll
        for (int v = 0; v < 3; ++v) w[v] = fr_const(f, r, v);
    } else if (f.first && idx >= f.n_s) {
        fr_ends(f, r, idx - f.n_s, w);
    } else {
#pragma unroll
        for (int v = 0; v < 3; ++v) w[v] = f.A[v * f.a_stride + r.col + idx];
    }
}

struct FrLds {
    Coef c[16];
    double box[2];
    int bad;
    double F[3][kFrNs];     // point fluxes
    double Fs[2][3];        // common fluxes at the two faces
    double w[3][16];        // updated element: solution points, then end values
};

// The residual and the stage update of element e by one wave, into L.w.
__device__ __forceinline__ void fr_update(const FrStageArgs& f, int64_t e, int lane, FrLds& L) {
    // values on both sides of the two faces, lane 2 face + side
    const int q = lane & 3;
    const FrElem r = fr_elem(f, q == 0 ? e - 1 : q == 3 ? e + 1 : e);
    double s[3];
    if (r.ghost) {
#pragma unroll
        for (int v = 0; v < 3; ++v) s[v] = fr_const(f, r, v);
    } else {
        fr_ends(f, r, (q & 1) ^ 1, s);
    }
    double wl[3], wr[3], Fs[3];
#pragma unroll
    for (int v = 0; v < 3; ++v) {
        wl[v] = __shfl(s[v], 2 * (lane & 1), 64);
        wr[v] = __shfl(s[v], 2 * (lane & 1) + 1, 64);
    }
    fr_hllc(f.gamma, f.gm1, wl, wr, Fs);
    if (lane < 2)
#pragma unroll
        for (int v = 0; v < 3; ++v) L.Fs[lane][v] = Fs[v];
    // point fluxes, lane = solution point (zero past the last one)
    const int64_t c0 = e * f.n_v;
    if (lane < kFrNs) {
        double w[3], fx[3] = {0.0, 0.0, 0.0};
        if (lane < f.n_s) {
#pragma unroll
            for (int v = 0; v < 3; ++v) w[v] = f.A[v * f.a_stride + c0 + lane];
            fr_euler_flux(f.gm1, w, fx);
        }
#pragma unroll
        for (int v = 0; v < 3; ++v) L.F[v][lane] = fx[v];
    }
    wave_lds_fence();
    // residual and Shu-Osher combination, lane = (variable, solution point)
    const int v = lane >> 3, j = lane & 7;
    if (v < 3) {
        double F[kFrNs];
#pragma unroll
        for (int k = 0; k < kFrNs; ++k) F[k] = L.F[v][k];
        const double jl = L.Fs[0][v] - fr_end_dot(f, 0, F);
        const double jr = L.Fs[1][v] - fr_end_dot(f, 1, F);
        double d = 0.0;
#pragma unroll
        for (int k = 0; k < kFrNs; ++k) d = fma(f.D[j][k], F[k], d);
        d = fma(jl, f.dg[0][j], d);
        d = fma(jr, f.dg[1][j], d);
        const double R = -f.inv_jac * d;
        const double dt = f.tdt ? f.tdt[1] : f.dt;
        double nu = 0.0;
        if (j < f.n_s) {
            const double x = f.A[v * f.a_stride + c0 + j];
            const double u0 = f.U0[v * f.u0_stride + c0 + j];
            nu = f.ca * u0 + f.cb * (x + dt * R);
            L.w[v][j] = nu;
        }
        // end values of the update: each lane of a variable holds all points
        double u[kFrNs];
#pragma unroll
        for (int k = 0; k < kFrNs; ++k) u[k] = __shfl(nu, (lane & ~7) + k, 64);
        if (j < 2) L.w[v][f.n_s + j] = fr_end_dot(f, j, u);
    }
}

template <int NT, int T>
__global__ __launch_bounds__(NT) void fr1d_stage_limited(FrStageArgs f) {
    constexpr int NW = NT / 64;
    constexpr int kRhsWave = NW > 1 ? 1 : 0, kLimWave = NW > 2 ? 2 : 0;
    __shared__ ExpPair sExp[256];
    __shared__ Red red;
    __shared__ FrLds L;
    const BoundsArgs& p = f.b;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t e = xcd_range(f.n_launch, 0).e;
    const bool ghost = e >= f.n_elem;      // a Dirichlet ghost element (last stage)
    const int S = ghost ? f.n_v : f.n_v + 2;
    stage_exp_table<NT>(sExp);
    if (wid == 0) {
        double lo = kInf, hi = -kInf;
        bool ok = true;
        if (lane < S) {
            double w[3];
            if (ghost) {
#pragma unroll
                for (int v = 0; v < 3; ++v) w[v] = e == f.n_elem ? f.left[v] : f.right[v];
            } else {
                stencil_state(f, e, lane, w);
            }
            const Prim st = make_prim<1>(p, w[0], w[1], 0.0, 0.0, w[2]);
            ok = st.ok;
            if (ok) {
                const double lt = log(2.0 * kPi * st.th);
                const double a = log(st.rho) - 0.5 * lt;
                // ln(theta delta / 2) from the same log
                L.c[lane] = Coef{a, p.half_delta > 0.0 ? a + (lt + f.lhd) : -kInf, st.ux, 0.0,
                                 -0.5 / st.th};
                const double sd = sqrt(st.th);
                lo = box_lo(st.ux, p.k, sd);
                hi = box_hi(st.ux, p.k, sd);
            }
        }
        const bool bad = __builtin_amdgcn_ballot_w64(!ok) != 0;
        lo = limiter::grp_min<16>(lo);
        hi = limiter::grp_max<16>(hi);
        if (lane == 0) {
            L.box[0] = p.grid_mode == KBL_GRID_STENCIL ? lo : p.lo0;
            L.box[1] = p.grid_mode == KBL_GRID_STENCIL ? hi : p.hi0;
            L.bad = bad;
        }
    }
    if (wid == kRhsWave) {
        if (!ghost) {
            fr_update(f, e, lane, L);
        } else if (lane < f.n_v) {
#pragma unroll
            for (int v = 0; v < 3; ++v) L.w[v][lane] = e == f.n_elem ? f.left[v] : f.right[v];
        }
    }
    __syncthreads();
    const bool bad = L.bad != 0;
    if (!bad) {
        const double lo = L.box[0];
        const double h = (L.box[1] - lo) / (double)(p.nx - 1);
        Sums1D sums;
        for (int j0 = 0; j0 < p.nx; j0 += NT * T) {
            Env1D<T> env;
            env.fold(p, L.c, S, lo, h, j0 + tid, NT, true);
            env.contract(p, lo, h, j0 + tid, NT, sExp, sums);
        }
        double part[8];
        sums.parts(1.0 - p.r_fac, 1.0 + p.r_fac, part);
        const double y = wave_transpose8<OpSum>(part);
        if ((lane & 7) == 0) red.v[wid][lane >> 3] = y;
    }
    __syncthreads();
    if (wid != kLimWave) return;
    // limiter, lane = node (the wave's four groups of 16 lanes do the same)
    double b[6];
    bool bad_b = bad;
    if (!bad) {
        double sum[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            sum[i] = red.v[0][i];
#pragma unroll
            for (int w = 1; w < NW; ++w) sum[i] += red.v[w][i];
        }
        b[0] = sum[0] < p.rho_floor ? p.rho_floor : sum[0];
        b[3] = sum[1];
        b[2] = sum[2];
        b[5] = sum[3];
        b[1] = sum[4];
        b[4] = sum[5];
#pragma unroll
        for (int i = 0; i < 6; ++i) bad_b |= !finite_bits(b[i]);
    } else {
#pragma unroll
        for (int i = 0; i < 6; ++i) b[i] = 0.0;
    }
    const int j = lane & 15;
    const bool live = j < f.n_v;
    double w[3], wt[3], amin, aP;
    uint32_t st;
#pragma unroll
    for (int v = 0; v < 3; ++v) w[v] = live ? L.w[v][j] : 0.0;
    limiter::limit_group<1, 16>(f.l, w, b, f.l.c[j], live, bad_b, wt, amin, aP, st);
    if (lane < f.n_v) {
#pragma unroll
        for (int v = 0; v < 3; ++v) f.B[v * f.b_stride + e * f.n_v + lane] = wt[v];
        if (lane == 0 && f.status) f.status[e] = st;
    }
}

template <int NT, int T>
hipError_t launch_stage_limited(const FrStageArgs& f, hipStream_t stream) {
    hipLaunchKernelGGL((fr1d_stage_limited<NT, T>), dim3((unsigned)f.n_launch), dim3(NT), 0,
                       stream, f);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fr1d_stage_limited(const FrStageArgs& f, hipStream_t stream) {
    if (f.b.nx <= 64) return launch_stage_limited<64, 1>(f, stream);
    if (f.b.nx <= 256) return launch_stage_limited<256, 1>(f, stream);
    return launch_stage_limited<256, 2>(f, stream);
}

}  // namespace kbl
