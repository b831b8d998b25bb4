// FP64 kinetic bounds in 2D with per-block culling of the stencil states
// (steps 1-3 of the overview in Sec. 3.9), gfx950.
//
// The envelopes of eq. fminmax take, at every velocity node, the largest and
// the smallest of the stencil's Maxwellians.  Few states ever win near a given
// node: over a block of a few nodes two or three out of 80 in most blocks, and
// many only in the blocks where the states are nearly tied.  The kernel
// therefore first decides, block by block, which states can win at all, and
// evaluates only those.  What it leaves out is proven to be no extremum at any
// node of the block, so the envelopes are those of the full evaluation.
//
// One wave owns one element; the four waves of a workgroup are independent and
// share the exp table (one workgroup per element, with barriers between the
// steps, ran 1.5 times slower: three elements in flight per CU instead of
// twelve do not cover the latency of the steps).  The velocity grid is cut
// into at most 8 x 8 blocks of bw x bh nodes (bw, bh even, 2 to 8).
//  1. Prologue, lane = state: admissibility, log-Maxwellian coefficients
//       q_i(u) = a_i + nk_i |u - U_i|^2,  a = ln rho - ln(2 pi theta),
//       nk = -1 / (2 theta),  l = ln(theta delta / 2),
//     staged in LDS, and the velocity box of eq. truncdomain.
//  2. Cull, lane = block, two loops over the states.  The first finds the
//     state r+ (r-) whose q is largest (smallest) at the block's centre, up to
//     2^-44 of its value (in FP32, up to 2^-15, flows that vary less within a
//     stencil had arbitrary references and kept most states: 40000 quads of 80
//     states that differ by 1e-6 took 4.0 ms on 64 x 64 nodes, 1.9 now).  The
//     second bounds q_i - q_r over the block: with the half widths wx, wy and
//     the gradients 2 nk (c - U) at the centre c,
//       q_i - q_r <= (q_i - q_r)(c) + wx |dgx| + wy |dgy|
//                    + (wx^2 + wy^2) max(nk_i - nk_r, 0),
//     and a state whose bound, raised by max(l_i - l_r, 0) for the internal
//     part g_I = e^l g (Sec. 3.6), is negative beats r+ nowhere in the block in
//     either envelope; likewise from below for r-.  The survivors' indices
//     go to a list per block and side; a list that would not fit its row
//     stands for all states.
//  3. The blocks are sorted by the length of their lists (six stable radix
//     passes over the lanes), so that the blocks a wave evaluates together
//     have lists of nearly the same length.
//  4. Evaluation: (bw / 2)(bh / 2) lanes per block, 2 x 2 nodes per lane,
//     64 / that many blocks per pass: the upper, then the lower envelopes of g and g_I in the log domain (where
//     the lists are long, all states and both sides at once), one exp per
//     node and envelope, and the moment contraction (eq. rhobounds, Ebounds,
//     mmbounds, mpbounds) with trapezoid weights (Sec. 3.7).
//  5. One reduction over the wave, relaxation (eq. relaxed), floor, store.
// The order of all sums is fixed: results are bitwise deterministic.
//
// What bounds it: VALU issue (88% busy at three waves per SIMD; these are the
// counters of the case tri_1000, kept under profiles/).  Two million triangles on
// a 64 x 64 grid take 67.4 ms against 147.4 ms for evaluating every pair
// (bounds_fp64_2d), 16.8k VALU instructions per element against 39.7k: the cull
// 3.8k, 16 passes of about 430 besides the list states, 35 per list step.  With
// the limiter, 512^2 quads on a global 64 x 64 grid take 8.6 against 19.0 ms;
// 256^2 quads on a 48 x 48 per-stencil grid, whose blocks near ties keep long
// lists, 2.80 against 3.20 ms with the limiter and the backward (85% busy).  At
// three waves 110 values wait in scratch outside the inner loops: 88 GB per launch
// on the triangles, 1.3 TB/s, a third of a copy's rate.  Four waves per SIMD (128
// VGPRs) spilled in the loops and ran 25% slower.
// Where it loses: states that tie up to rounding but are not equal (a uniform
// flow after a few steps).  No block can leave out any, and q is formed for 2 x 2
// nodes at a time: 40000 quads of 80 such states take 4.2 ms against 2.95.
//
// Rounding: the bounds of step 2 are computed in FP64, half widths widened by 1e-10
// and thresholds by 1e-12 relative, far above their rounding error.
#include <type_traits>

#include "bounds_common.h"

namespace kbl {
namespace {

constexpr int kCullRow = 32;       // list entries per block and side

struct CullGrid {
    int hw, hh;          // lanes per block in x and y: blocks of 2 hw x 2 hh nodes
    uint32_t inv_ns;     // ceil(2^32 / n_s) for n_s > 1
    double lhd;          // ln(delta / (4 pi)); 0 without internal degrees of freedom
};

// One stencil state: q = a + nk ((ux - U_x)^2 + (uy - U_y)^2), q_I = q + l.
struct CullRec {
    double a, l, ux, uy, nk;
};

// Velocity node of one direction: position and trapezoid weight (0 past the
// grid, where the position repeats the last node).
struct alignas(16) CullNode {
    double u, w;
};
constexpr int kCullNodes = 64 + 2;   // two more of weight 0, for idle lanes

struct CullLds {
    CullRec rec[kCullCap];
    uint8_t list[2][64][kCullRow];
    uint8_t all[kCullCap];
    CullNode node[2][kCullNodes];
};

// The wave's own LDS accesses execute in program order; this only keeps the
// compiler from moving accesses of other lanes' data across it.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ double read_lane_f64(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readlane((int)b, lane);
    const unsigned hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | lo);
}

// Loads state s of the row and forms its record.  inv_ns = ceil(2^32 / n_s)
// (n_s > 1): s / n_s is exact for s, n_s < 2^16.  Returns 0 or a status bit.
struct CullState {
    CullRec r;
    double th;
};
__device__ __forceinline__ uint32_t cull_state(const BoundsArgs& p, int64_t row0, int s,
                                               uint32_t inv_ns, double lhd, CullState* out) {
    int unit = s;
    if (p.n_s > 1) unit = s < 65536 ? (int)__umulhi((unsigned)s, inv_ns) : s / p.n_s;
    const int32_t col = p.cols[row0 + unit];
    if (col < 0 || col >= p.n_src) return KBL_ST_BAD_STENCIL;
    const Prim st = load_prim<2>(p, (int64_t)col * p.n_s + (s - unit * p.n_s));
    if (!st.ok) return KBL_ST_INADMISSIBLE;
    const double lt = log(2.0 * kPi * st.th);
    out->r.a = log(st.rho) - lt;
    out->r.l = lt + lhd;              // ln(theta delta / 2)
    out->r.ux = st.ux;
    out->r.uy = st.uy;
    out->r.nk = -0.5 / st.th;
    out->th = st.th;
    return 0;
}

__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(3))) void bounds_cull_2d(BoundsArgs p, CullGrid cg) {
    __shared__ ExpPair sExp[256];
    __shared__ CullLds lds[kWaves];
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    CullLds& L = lds[wid];
    stage_exp_table<kThreads>(sExp);
    for (int j = lane; j < kCullCap; j += 64) L.all[j] = (uint8_t)j;
    __syncthreads();

    const double rm = 1.0 - p.r_fac, rp = 1.0 + p.r_fac;
    const double has_int = p.half_delta > 0.0 ? 1.0 : 0.0;
    // evaluation: lane -> (block of the pass, 2 x 2 nodes in the block)
    const int lpt = cg.hw * cg.hh;
    const int grp = lane / lpt;
    const int pos = lane - grp * lpt;
    const int py = pos / cg.hw, px = pos - py * cg.hw;
    const int per_pass = 64 / lpt;
    // cull: lane -> block
    const int bx = lane & 7, by = lane >> 3;
    const bool is_block = bx * 2 * cg.hw < p.nx && by * 2 * cg.hh < p.ny;
    const int n_blocks = __popcll(__ballot(is_block));

    ElemRange er = xcd_range(p.n_elem, p.grid_blocks);
    for (er.e += wid * er.step; er.e < er.end; er.e += kWaves * er.step) {
        const int64_t e = er.e;
        const int64_t row0 = p.rowptr[e], row1 = p.rowptr[e + 1];
        if (row0 < 0 || row1 <= row0 || row1 > p.nnz) {
            if (lane == 0) store_nan<2>(p, e, KBL_ST_BAD_STENCIL);
            continue;
        }
        int S = (int)(row1 - row0) * p.n_s;

        // ---- 1. prologue
        uint32_t bad = 0;
        bool cold = false;
        double ext[8] = {kInf, kInf, kInf, kInf, 0.0, 0.0, 0.0, 0.0};
        for (int s = lane; s < S; s += 64) {
            CullState st;
            const uint32_t b = cull_state(p, row0, s, cg.inv_ns, cg.lhd, &st);
            bad |= b;
            if (b) continue;
            if (s < kCullCap) L.rec[s] = st.r;
            cold |= !finite_bits(st.r.nk);
            const double sd = sqrt(st.th);
            ext[0] = fmin(ext[0], box_lo(st.r.ux, p.k, sd));
            ext[1] = fmin(ext[1], -box_hi(st.r.ux, p.k, sd));
            ext[2] = fmin(ext[2], box_lo(st.r.uy, p.k, sd));
            ext[3] = fmin(ext[3], -box_hi(st.r.uy, p.k, sd));
        }
        if (__ballot(bad != 0)) {
            // a bad row is reported alone (its other states are not a stencil)
            const uint32_t f = __ballot((bad & KBL_ST_BAD_STENCIL) != 0) ? KBL_ST_BAD_STENCIL
                                                                        : KBL_ST_INADMISSIBLE;
            if (lane == 0) store_nan<2>(p, e, f);
            continue;
        }
        double lox = p.lo0, hix = p.hi0, loy = p.lo1, hiy = p.hi1;
        if (p.grid_mode == KBL_GRID_STENCIL) {
            const double m = wave_transpose8<OpMin>(ext);
            lox = read_lane_f64(m, 0);
            hix = -read_lane_f64(m, 8);
            loy = read_lane_f64(m, 16);
            hiy = -read_lane_f64(m, 24);
        }
        const double hx = (hix - lox) / (double)(p.nx - 1);
        const double hy = (hiy - loy) / (double)(p.ny - 1);
        const bool big = S > kCullCap;
        // no bounds of q without a finite nk (a denormal temperature)
        const bool all = big || __ballot(cold) != 0;
        // velocity nodes and trapezoid weights
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const int n = d ? p.ny : p.nx;
            const double lo = d ? loy : lox, h = d ? hy : hx;
            CullNode t;
            t.u = node_pos(lo, lane < n ? lane : n - 1, h);
            t.w = lane < n ? h * ((lane == 0 || lane == n - 1) ? 0.5 : 1.0) : 0.0;
            L.node[d][lane] = t;
            if (lane < 2) L.node[d][64 + lane] = CullNode{t.u, 0.0};
        }
        wave_lds_fence();

        // ---- 2. cull: lane = block
        int cm = 0, cn = 0;              // list lengths: upper, lower envelopes; 0: all states
        if (!all) {
            const int x0 = bx * 2 * cg.hw, y0 = by * 2 * cg.hh;
            const double xa = L.node[0][x0 < 64 ? x0 : 63].u;
            const double xb = L.node[0][x0 + 2 * cg.hw - 1 < 64 ? x0 + 2 * cg.hw - 1 : 63].u;
            const double ya = L.node[1][y0 < 64 ? y0 : 63].u;
            const double yb = L.node[1][y0 + 2 * cg.hh - 1 < 64 ? y0 + 2 * cg.hh - 1 : 63].u;
            const double cx = 0.5 * (xa + xb), cy = 0.5 * (ya + yb);
            // twice the half widths (the gradient below is halved), widened
            const double wx = (xb - xa) * (1.0 + 1e-10) + 1e-14 * (fabs(xa) + fabs(xb));
            const double wy = (yb - ya) * (1.0 + 1e-10) + 1e-14 * (fabs(ya) + fabs(yb));
            const double Q = 0.25 * (wx * wx + wy * wy);
            double kmax = -kInf, kmin = kInf;
#pragma unroll 4
            for (int s = 0; s < S; ++s) {
                const CullRec& r = L.rec[s];
                const double dx = cx - r.ux, dy = cy - r.uy;
                const double v = fma(r.nk, fma(dx, dx, dy * dy), r.a);
                // the state's index in the low byte (any state is a valid reference)
                const double key = __hiloint2double(__double2hiint(v), (__double2loint(v) & ~255) | s);
                kmax = fmax(kmax, key);
                kmin = fmin(kmin, key);
            }
            double vr[2], tr[2], sr[2], lr[2], qr[2];
            double slacks = 0.0;
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const int ref = __double2loint(side ? kmin : kmax) & 127;
                const CullRec r = L.rec[ref];
                const double dx = cx - r.ux, dy = cy - r.uy;
                tr[side] = r.nk * dx;
                sr[side] = r.nk * dy;
                const double v = fma(tr[side], dx, fma(sr[side], dy, r.a));
                qr[side] = Q * r.nk;
                const double slack = 1e-12 * (1.0 + fabs(v) + fabs(r.a) + wx * fabs(tr[side]) +
                                              wy * fabs(sr[side]) + fabs(qr[side]) + fabs(r.l));
                slacks += slack;
                lr[side] = r.l;
                vr[side] = (side ? v + slack : v - slack) + (r.l + qr[side]);
            }
            uint8_t* const row0p = L.list[0][lane];
            uint8_t* const row1p = L.list[1][lane];
#pragma unroll 4
            for (int s = 0; s < S; ++s) {
                const CullRec& r = L.rec[s];
                const double dx = cx - r.ux, dy = cy - r.uy;
                const double t = r.nk * dx, u = r.nk * dy, qn = Q * r.nk;
                const double v = fma(t, dx, fma(u, dy, r.a));
                // max(l - l_r, 0) + max(qn - qn_r, 0), with l_r + qn_r in vr
                const double up = fma(wx, fabs(t - tr[0]), fma(wy, fabs(u - sr[0]),
                                      (v - vr[0]) + (fmax(r.l, lr[0]) + fmax(qn, qr[0]))));
                const double dn = fma(-wx, fabs(t - tr[1]), fma(-wy, fabs(u - sr[1]),
                                      (v - vr[1]) + (fmin(r.l, lr[1]) + fmin(qn, qr[1]))));
                const bool au = up >= 0.0, an = dn <= 0.0;
                if (au) row0p[cm < kCullRow ? cm : kCullRow - 1] = (uint8_t)s;
                cm += au ? 1 : 0;
                if (an) row1p[cn < kCullRow ? cn : kCullRow - 1] = (uint8_t)s;
                cn += an ? 1 : 0;
            }
            const bool finite = finite_bits(slacks);
            cm = finite ? cm : 0;
            cn = finite ? cn : 0;
            if (__ballot(cm + cn < 2 * S) == 0) {
                // Every block keeps every state: they may all be the same, as in a
                // constant field, and the first then stands for all (40000 quads of 80
                // equal states on 64 x 64 nodes: 0.93 ms, 4.3 with all evaluated).
                const CullRec f = L.rec[0];
                bool differs = false;
                for (int s = lane; s < S; s += 64) {
                    const CullRec r = L.rec[s];
                    differs |= r.a != f.a || r.l != f.l || r.ux != f.ux || r.uy != f.uy || r.nk != f.nk;
                }
                if (__ballot(differs) == 0) {
                    S = 1;
                    cm = 0;
                    cn = 0;
                }
            }
        }

        // ---- 3. blocks in ascending order of list length
        const int em = cm == 0 || cm > kCullRow ? S : cm, en = cn == 0 || cn > kCullRow ? S : cn;
        int order;                       // lane i: block and lengths at place i
        {
            int key = em + en;
            key = key < 32 ? key : (32 + (key - 32) / 8 < 63 ? 32 + (key - 32) / 8 : 63);
            if (!is_block) key = 0;      // sorted first (real blocks have key >= 2)
            if (all) key = is_block ? 1 : 0;
            unsigned v = (unsigned)key | ((unsigned)lane << 6) |
                         ((unsigned)(cm > kCullRow ? 0 : cm) << 12) |
                         ((unsigned)(cn > kCullRow ? 0 : cn) << 20);
            static_assert(kCullRow < 256, "list lengths take 8 bits");
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                const bool one = (v >> b) & 1u;
                const unsigned long long ones = __ballot(one);
                const int before = __builtin_amdgcn_mbcnt_hi(
                    (unsigned)(ones >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)ones, 0));
                const int to = one ? 64 - __popcll(ones) + before : lane - before;
                v = (unsigned)__builtin_amdgcn_ds_permute(to << 2, (int)v);
            }
            order = (int)v;
        }
        wave_lds_fence();

        // ---- 4. evaluation
        // sums over the unrelaxed envelopes: rho, E (lower, upper), momentum
        // split by the sign of u (see the contraction below)
        double s_rho[2] = {0, 0}, s_e[2] = {0, 0}, s_ei[2] = {0, 0};   // s_e: of |u|^2 g
        double s_neg[2][2] = {{0, 0}, {0, 0}}, s_pos[2][2] = {{0, 0}, {0, 0}};   // [envelope][dir]
        for (int b0 = 64 - n_blocks; b0 < 64; b0 += per_pass) {
            const int slot = b0 + grp;
            const bool act = slot < 64 && grp < per_pass;
            const unsigned o = (unsigned)__builtin_amdgcn_ds_bpermute((slot < 64 ? slot : 63) << 2, order);
            const int blk = (o >> 6) & 63;
            // idle lanes take nodes of weight 0
            const int jx = act ? (blk & 7) * 2 * cg.hw + 2 * px : 64;
            const int jy = (blk >> 3) * 2 * cg.hh + 2 * py;
            double x[2], y[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                x[i] = L.node[0][jx + i].u;
                y[i] = L.node[1][jy + i].u;
            }
            // the longest lists of the pass are those of its last block
            const unsigned last = __builtin_amdgcn_readlane(order, b0 + per_pass < 64 ? b0 + per_pass - 1 : 63);
            const int lm = (last >> 12) & 255, ln = (last >> 20) & 255;
            const bool dual = big || 30 * ((lm ? lm : S) + (ln ? ln : S)) > 38 * S;
            double qx[2][2], qix[2][2], qn[2][2], qin[2][2];   // upper, lower envelopes of q, q_I
            auto values = [&](const CullRec& r, double (&v)[2][2]) {
                double A[2], Y[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const double dx = x[i] - r.ux, dy = y[i] - r.uy;
                    A[i] = fma(r.nk * dx, dx, r.a);
                    Y[i] = dy * dy;
                }
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) v[i][j] = fma(r.nk, Y[j], A[i]);
            };
            if (!dual) {
                // one side after the other over the block's lists
                auto side = [&](auto up_t, double (&q)[2][2], double (&qi)[2][2]) {
                    constexpr bool UP = decltype(up_t)::value;
                    int n = (o >> (UP ? 12 : 20)) & 255;
                    const uint8_t* lst = n ? L.list[UP ? 0 : 1][blk] : L.all;
                    const int lim = (n ? n : S) - 1;
                    n = !act ? 1 : n ? n : S;
                    // the next state's record and the index after it are read
                    // before the current state's work; past its own list a
                    // block repeats its last state
                    const uint8_t* const end = lst + lim;
                    auto next = [&]() {
                        const int i = *lst;
                        lst = lst < end ? lst + 1 : end;
                        return i;
                    };
                    auto take = [&](const CullRec& r) {
                        double v[2][2];
                        values(r, v);
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                const double vi = v[i][j] + r.l;
                                q[i][j] = UP ? fmax(q[i][j], v[i][j]) : fmin(q[i][j], v[i][j]);
                                qi[i][j] = UP ? fmax(qi[i][j], vi) : fmin(qi[i][j], vi);
                            }
                    };
                    CullRec ra = L.rec[next()];
                    int nx = next();
                    CullRec rb = L.rec[nx];
                    nx = next();
                    {
                        double v[2][2];
                        values(ra, v);
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                q[i][j] = v[i][j];
                                qi[i][j] = v[i][j] + ra.l;
                            }
                    }
                    int k = 1;
                    if (__builtin_amdgcn_ballot_w64(k < n)) {
                        do {
                            ra = rb;
                            rb = L.rec[nx];
                            nx = next();
                            take(ra);
                            ++k;
                        } while (__builtin_amdgcn_ballot_w64(k < n));
                    }
                };
                side(std::true_type{}, qx, qix);
                side(std::false_type{}, qn, qin);
            } else {
                // long lists: all states, both sides at once.  Stencils
                // beyond the staged states go chunk by chunk, staged again
                // for every pass.
                for (int c0 = 0; c0 < S; c0 += kCullCap) {
                    const int cnt = S - c0 < kCullCap ? S - c0 : kCullCap;
                    if (big) {
                        wave_lds_fence();
                        for (int s = lane; s < cnt; s += 64) {
                            CullState st;
                            (void)cull_state(p, row0, c0 + s, cg.inv_ns, cg.lhd, &st);
                            L.rec[s] = st.r;
                        }
                        wave_lds_fence();
                    }
                    if (c0 == 0) {
                        const CullRec r = L.rec[0];
                        values(r, qx);
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                qn[i][j] = qx[i][j];
                                qix[i][j] = qin[i][j] = qx[i][j] + r.l;
                            }
                    }
#pragma unroll 2
                    for (int s = c0 == 0 ? 1 : 0; s < cnt; ++s) {
                        const CullRec r = L.rec[s];
                        double v[2][2];
                        values(r, v);
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                const double vi = v[i][j] + r.l;
                                qx[i][j] = fmax(qx[i][j], v[i][j]);
                                qn[i][j] = fmin(qn[i][j], v[i][j]);
                                qix[i][j] = fmax(qix[i][j], vi);
                                qin[i][j] = fmin(qin[i][j], vi);
                            }
                    }
                }
            }
            // exps of a pair of nodes in three phases (indices and
            // polynomials, the table reads together, the products), and the
            // separable contraction M = wx wy: row sums over y, column sums
            // over x
            double wx[2], wy[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                wx[i] = L.node[0][jx + i].w;
                wy[i] = L.node[1][jy + i].w;
            }
            auto contract = [&](auto up_t, const double (&q)[2][2], const double (&qi)[2][2]) {
                double r0[2] = {0, 0}, c0[2] = {0, 0}, ri = 0.0;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    ExpPrep pr[4];
                    ExpPair T[4];
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        pr[2 * j] = exp_prep(q[i][j]);
                        pr[2 * j + 1] = exp_prep(qi[i][j]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int k = 0; k < 4; ++k) T[k] = sExp[pr[k].ni & 255];
                    __builtin_amdgcn_sched_barrier(0);
                    double t = 0.0;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const double g = exp_fin(pr[2 * j], T[2 * j]);
                        const double gi = exp_fin(pr[2 * j + 1], T[2 * j + 1]);
                        r0[i] = fma(wy[j], g, r0[i]);
                        c0[j] = fma(wx[i], g, c0[j]);
                        t = fma(wy[j], gi, t);
                    }
                    ri = fma(wx[i], t, ri);
                    __builtin_amdgcn_sched_barrier(0);
                }
                constexpr int d = decltype(up_t)::value ? 1 : 0;
                s_rho[d] = fma(wx[0], r0[0], s_rho[d]);
                s_rho[d] = fma(wx[1], r0[1], s_rho[d]);
                s_ei[d] += ri;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const double mux = wx[i] * x[i], muy = wy[i] * y[i];
                    s_e[d] = fma(mux * x[i], r0[i], s_e[d]);
                    s_e[d] = fma(muy * y[i], c0[i], s_e[d]);
                    s_neg[d][0] = fma(fmin(mux, 0.0), r0[i], s_neg[d][0]);
                    s_pos[d][0] = fma(fmax(mux, 0.0), r0[i], s_pos[d][0]);
                    s_neg[d][1] = fma(fmin(muy, 0.0), c0[i], s_neg[d][1]);
                    s_pos[d][1] = fma(fmax(muy, 0.0), c0[i], s_pos[d][1]);
                }
            };
            contract(std::true_type{}, qx, qix);
            contract(std::false_type{}, qn, qin);
        }

        // ---- 5. reduction, relaxation, store.  Momentum (eq. mmbounds,
        // mpbounds): the lower bound takes the upper envelope where u < 0 and
        // the lower one where u >= 0, the upper bound the reverse.
        double part[8] = {rm * s_rho[0], rp * s_rho[1], rm * fma(0.5, s_e[0], has_int * s_ei[0]),
                          rp * fma(0.5, s_e[1], has_int * s_ei[1]),
                          rp * s_neg[1][0] + rm * s_pos[0][0], rm * s_neg[0][0] + rp * s_pos[1][0],
                          rp * s_neg[1][1] + rm * s_pos[0][1], rm * s_neg[0][1] + rp * s_pos[1][1]};
        const double sum = wave_transpose8<OpSum>(part);
        if ((lane & 7) == 0) store_bound_value<2>(p, e, lane >> 3, sum, 0);
        wave_lds_fence();
    }
}

}  // namespace

// Grids of up to 64 x 64 nodes; state indices of a row in 32 bits.
bool bounds_cull_fits(const BoundsArgs& a) {
    return a.nx <= 64 && a.ny <= 64 && a.n_s < 65536 && a.nnz <= (int64_t)INT32_MAX / a.n_s;
}

hipError_t launch_bounds_cull_2d(const BoundsArgs& a, hipStream_t stream) {
    if (!bounds_cull_fits(a)) return hipErrorInvalidValue;
    CullGrid g;
    g.hw = (a.nx + 15) / 16;
    g.hh = (a.ny + 15) / 16;
    g.inv_ns = a.n_s > 1 ? (uint32_t)(((1ull << 32) + a.n_s - 1) / a.n_s) : 0;
    g.lhd = a.half_delta > 0.0 ? log(a.half_delta) - log(2.0 * kPi) : 0.0;
    // k elements per workgroup of the other kernels are k per wave here
    BoundsArgs b = a;
    if (a.grid_blocks <= 0 && a.grid_blocks > -(int64_t)INT32_MAX)
        b.grid_blocks = kWaves * (a.grid_blocks ? a.grid_blocks : -1);
    hipLaunchKernelGGL(bounds_cull_2d, dim3(bounds_grid(b)), dim3(kThreads), 0, stream, b, g);
    return hipGetLastError();
}

}  // namespace kbl
