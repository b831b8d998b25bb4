// FP64 kinetic bounds over a three-dimensional velocity grid with per-block
// culling of the stencil states (steps 1-3 of the overview in Sec. 3.9), gfx950.
//
// The method is that of the 2D culling kernel (bounds_cull_2d.hip): over a
// block of velocity nodes few of the stencil's Maxwellians can be the largest
// or the smallest, the others are excluded by bounding q_i - q_r over the block
// against the state r that is extreme at its centre, and only the rest is
// evaluated.  (4096 hexahedra of 189 states that differ by 1e-6 take 1.46 ms on
// 24^3 nodes, 3.26 with r found in FP32.)  Here q_i(u) = a_i + nk_i |u - U_i|^2 in three directions,
// a = ln rho - (3/2) ln(2 pi theta).
//
// One workgroup of four waves owns one element at a time.  The states' records
// are shared; the blocks (4 nodes per direction up to 32 nodes, else 8; at
// most 8 blocks per direction) are culled with one lane per block, 256 to a
// round, sorted by the length of their lists, and evaluated 2 x 2 x 2 nodes per
// lane, the passes dealt to the waves by their work.  One reduction per
// element.  The order of all sums is fixed: results are bitwise deterministic.
//
// Why blocks of 4: on 24^3 nodes and stencils of 189 states the lists hold
// 15-20 states per side on average (3-4 in the median block) against 43-52
// for blocks of 6 nodes, whose cull costs a quarter.
//
// What bounds it: VALU issue and latency (80% busy at three waves per SIMD, by the
// counters of the case hex_32 kept under profiles/; 154k VALU instructions per element on 24^3 nodes
// and 189 states, against 294k for every pair).  32^3 hexahedra with the limiter:
// 10.5 against 17.7 ms (bounds_fp64_3d).  States that tie up to rounding but are
// not equal are all evaluated: 4096 hexahedra 3.1 against 2.25 ms.  Values kept in
// scratch outside the list loops move 9.8 GB per launch of 32^3 (0.9 TB/s).
// Sorting all blocks of an element instead of each wave's own, and dealing
// the passes by their work, took it from 12.3 to 11.7 ms; list addresses kept
// out of scratch from 11.7 to 11.0 ms.
//
// Rounding: half widths are widened by 1e-10 and thresholds by 1e-12 relative, far
// above the rounding error of the FP64 bounds.
#include "bounds_common.h"

namespace kbl {
namespace {

constexpr int kCap = kCullCap3;  // states staged at once
constexpr int kRow = 56;         // list entries per block and side

struct CullGrid3 {
    int hb[3];           // lanes per block and direction: blocks of 2 hb nodes
    int nb[3];           // blocks per direction
    uint32_t inv_ns;     // ceil(2^32 / n_s) for n_s > 1
    double lhd;          // ln(delta / (4 pi)); 0 without internal degrees of freedom
};

// One stencil state: q = a + nk |u - U|^2, q_I = q + l.
struct alignas(16) Rec3 {
    double a, l, ux, uy, uz, nk;
};

// Velocity node of one direction: position and trapezoid weight (0 past the
// grid, where the position repeats the last node).
struct alignas(16) Node {
    double u, w;
};
constexpr int kNodes = 64 + 2;   // two more of weight 0, for idle lanes

constexpr int kSlots = 64 * kWaves;   // blocks of one round

// Flag beside the status bits of a stencil: a state without a finite nk (a
// denormal temperature), whose q has no bounds.
constexpr uint32_t kCold = 1u << 31;

struct Lds3 {
    Rec3 rec[kCap];
    uint8_t list[2][kSlots][kRow];
    uint8_t all[kCap];
    Node node[3][kNodes];
    unsigned comp[kSlots], order[kSlots], coord[kSlots];
};

__device__ __forceinline__ uint32_t cull_state3(const BoundsArgs& p, int64_t row0, int s,
                                                uint32_t inv_ns, double lhd, Rec3* r, double* th) {
    int unit = s;
    if (p.n_s > 1) unit = s < 65536 ? (int)__umulhi((unsigned)s, inv_ns) : s / p.n_s;
    const int32_t col = p.cols[row0 + unit];
    if (col < 0 || col >= p.n_src) return KBL_ST_BAD_STENCIL;
    const Prim st = load_prim<3>(p, (int64_t)col * p.n_s + (s - unit * p.n_s));
    if (!st.ok) return KBL_ST_INADMISSIBLE;
    const double lt = log(2.0 * kPi * st.th);
    r->a = log(st.rho) - 1.5 * lt;
    r->l = lt + lhd;                  // ln(theta delta / 2)
    r->ux = st.ux;
    r->uy = st.uy;
    r->uz = st.uz;
    r->nk = -0.5 / st.th;
    *th = st.th;
    return 0;
}

__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(3))) void bounds_cull_3d(BoundsArgs p, CullGrid3 cg) {
    __shared__ ExpPair sExp[256];
    __shared__ Lds3 L;
    __shared__ Red red;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    stage_exp_table<kThreads>(sExp);     // published by the prologue's barriers
    L.all[tid] = (uint8_t)tid;

    const double has_int = p.half_delta > 0.0 ? 1.0 : 0.0;
    // evaluation: lane -> (block of the pass, 2 x 2 x 2 nodes in the block)
    const int hx_ = cg.hb[0], hxy = cg.hb[0] * cg.hb[1], lpt = hxy * cg.hb[2];
    const int grp = lane / lpt, pos = lane - grp * lpt;
    const int pz = pos / hxy, pxy = pos - pz * hxy, py = pxy / hx_, px = pxy - py * hx_;
    const int per_pass = 64 / lpt;
    // groups of blocks: rounds of one group per wave, all of the same size
    const int n_blocks = cg.nb[0] * cg.nb[1] * cg.nb[2];
    const int rounds = (n_blocks + 64 * kWaves - 1) / (64 * kWaves);
    const int gsize = (n_blocks + kWaves * rounds - 1) / (kWaves * rounds);

    for (ElemRange er = xcd_range(p.n_elem, p.grid_blocks); er.e < er.end; er.e += er.step) {
        const int64_t e = er.e;
        const int64_t row0 = p.rowptr[e], row1 = p.rowptr[e + 1];
        if (row0 < 0 || row1 <= row0 || row1 > p.nnz) {
            if (tid == 0) store_nan<3>(p, e, KBL_ST_BAD_STENCIL);
            continue;
        }
        const int S = (int)(row1 - row0) * p.n_s;

        // ---- prologue
        uint32_t bad = 0;
        bool cold = false;
        double ext[8] = {kInf, kInf, kInf, kInf, kInf, kInf, 0.0, 0.0};
        for (int s = tid; s < S; s += kThreads) {
            Rec3 r;
            double th;
            const uint32_t b = cull_state3(p, row0, s, cg.inv_ns, cg.lhd, &r, &th);
            bad |= b;
            if (b) continue;
            if (s < kCap) L.rec[s] = r;
            cold |= !finite_bits(r.nk);
            const double sd = sqrt(th);
            ext[0] = fmin(ext[0], box_lo(r.ux, p.k, sd));
            ext[1] = fmin(ext[1], -box_hi(r.ux, p.k, sd));
            ext[2] = fmin(ext[2], box_lo(r.uy, p.k, sd));
            ext[3] = fmin(ext[3], -box_hi(r.uy, p.k, sd));
            ext[4] = fmin(ext[4], box_lo(r.uz, p.k, sd));
            ext[5] = fmin(ext[5], -box_hi(r.uz, p.k, sd));
        }
        if (tid == 0) red.flags = 0;
        const double m = wave_transpose8<OpMin>(ext);
        if ((lane & 7) == 0) red.v[wid][lane >> 3] = m;
        __syncthreads();
        bad |= cold ? kCold : 0u;
        if (bad) atomicOr(&red.flags, bad);
        // velocity nodes and trapezoid weights: wave j forms direction j
        if (wid < 3) {
            double lo = wid == 0 ? p.lo0 : wid == 1 ? p.lo1 : p.lo2;
            double hi = wid == 0 ? p.hi0 : wid == 1 ? p.hi1 : p.hi2;
            if (p.grid_mode == KBL_GRID_STENCIL) {
                auto ext_min = [&](int j) {
                    return fmin(fmin(red.v[0][j], red.v[1][j]), fmin(red.v[2][j], red.v[3][j]));
                };
                lo = ext_min(2 * wid);
                hi = -ext_min(2 * wid + 1);
            }
            const int n = wid == 0 ? p.nx : wid == 1 ? p.ny : p.nz;
            const double h = (hi - lo) / (double)(n - 1);
            Node t;
            t.u = node_pos(lo, lane < n ? lane : n - 1, h);
            t.w = lane < n ? h * ((lane == 0 || lane == n - 1) ? 0.5 : 1.0) : 0.0;
            L.node[wid][lane] = t;
            if (lane < 2) L.node[wid][64 + lane] = Node{t.u, 0.0};
        }
        __syncthreads();
        const bool any_cold = (red.flags & kCold) != 0;
        uint32_t flags = red.flags & ~kCold;
        if (flags) {
            // a bad row is reported alone (its other states are not a stencil)
            if (flags & KBL_ST_BAD_STENCIL) flags = KBL_ST_BAD_STENCIL;
            if (tid == 0) store_nan<3>(p, e, flags);
            __syncthreads();             // red is reused
            continue;
        }
        const bool big = S > kCap;
        int n_all = S;                   // states that an empty list stands for
        const bool all = big || any_cold;

        // relaxed sums of this thread: rho, E, momentum per direction; [0]
        // lower, [1] upper bound
        double a_rho[2] = {0, 0}, a_e[2] = {0, 0}, a_m[3][2] = {{0, 0}, {0, 0}, {0, 0}};

        for (int rd = 0; rd < rounds; ++rd) {
            // lane = block: every fourth block of the round's range goes to
            // this wave (neighbouring blocks have lists of similar length);
            // idle lanes repeat the last block
            const int g0 = rd * kWaves * gsize + wid;
            const int left = (n_blocks - g0 + kWaves - 1) / kWaves;
            const int gn = g0 >= n_blocks ? 0 : left < gsize ? left : gsize;
            const int real = n_blocks - rd * kWaves * gsize < kWaves * gsize
                                 ? n_blocks - rd * kWaves * gsize : kWaves * gsize;
            int b[3];
            {
                int id = g0 + kWaves * (lane < gn ? lane : (gn ? gn - 1 : 0));
                if (id >= n_blocks) id = n_blocks - 1;
                b[0] = id % cg.nb[0];
                const int t = id / cg.nb[0];
                b[1] = t % cg.nb[1];
                b[2] = t / cg.nb[1];
            }
            // ---- cull
            int cm = 0, cn = 0;          // 0: all states
            if (!all) {
                double c[3], w[3], Q = 0.0;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const int i0 = b[d] * 2 * cg.hb[d], i1 = i0 + 2 * cg.hb[d] - 1;
                    const double ua = L.node[d][i0].u, ub = L.node[d][i1].u;
                    c[d] = 0.5 * (ua + ub);
                    // twice the half width (the gradient below is halved), widened
                    w[d] = (ub - ua) * (1.0 + 1e-10) + 1e-14 * (fabs(ua) + fabs(ub));
                    Q = fma(0.25 * w[d], w[d], Q);
                }
                double kmax = -kInf, kmin = kInf;
#pragma unroll 4
                for (int s = 0; s < S; ++s) {
                    const Rec3& r = L.rec[s];
                    const double dx = c[0] - r.ux, dy = c[1] - r.uy, dz = c[2] - r.uz;
                    const double v = fma(r.nk, fma(dx, dx, fma(dy, dy, dz * dz)), r.a);
                    // the state's index in the low byte (any state is a valid
                    // reference)
                    const double key = __hiloint2double(__double2hiint(v), (__double2loint(v) & ~255) | s);
                    kmax = fmax(kmax, key);
                    kmin = fmin(kmin, key);
                }
                double vr[2], tr[2][3], lr[2], qr[2];
                double slacks = 0.0;
#pragma unroll
                for (int sd = 0; sd < 2; ++sd) {
                    const Rec3 r = L.rec[__double2loint(sd ? kmin : kmax) & 255];
                    const double dx = c[0] - r.ux, dy = c[1] - r.uy, dz = c[2] - r.uz;
                    tr[sd][0] = r.nk * dx;
                    tr[sd][1] = r.nk * dy;
                    tr[sd][2] = r.nk * dz;
                    const double v = fma(tr[sd][0], dx, fma(tr[sd][1], dy, fma(tr[sd][2], dz, r.a)));
                    qr[sd] = Q * r.nk;
                    lr[sd] = r.l;
                    const double slack = 1e-12 * (1.0 + fabs(v) + fabs(r.a) + w[0] * fabs(tr[sd][0]) +
                                                  w[1] * fabs(tr[sd][1]) + w[2] * fabs(tr[sd][2]) +
                                                  fabs(qr[sd]) + fabs(r.l));
                    slacks += slack;
                    vr[sd] = (sd ? v + slack : v - slack) + (r.l + qr[sd]);
                }
                // the rows' addresses are formed here (through an empty asm
                // statement): hoisted out of the element loop they would be
                // reloaded from scratch at every append
                int ot = tid;
                asm volatile("" : "+v"(ot));
                uint8_t* const row_u = L.list[0][ot];
                uint8_t* const row_l = L.list[1][ot];
                cm = 0;
                cn = 0;
#pragma unroll 4
                for (int s = 0; s < S; ++s) {
                    const Rec3& r = L.rec[s];
                    const double dx = c[0] - r.ux, dy = c[1] - r.uy, dz = c[2] - r.uz;
                    const double tx = r.nk * dx, ty = r.nk * dy, tz = r.nk * dz, qn = Q * r.nk;
                    const double v = fma(tx, dx, fma(ty, dy, fma(tz, dz, r.a)));
                    // max(l - l_r, 0) + max(qn - qn_r, 0), with l_r + qn_r in vr
                    const double up =
                        fma(w[0], fabs(tx - tr[0][0]), fma(w[1], fabs(ty - tr[0][1]),
                        fma(w[2], fabs(tz - tr[0][2]),
                            (v - vr[0]) + (fmax(r.l, lr[0]) + fmax(qn, qr[0])))));
                    const double dn =
                        fma(-w[0], fabs(tx - tr[1][0]), fma(-w[1], fabs(ty - tr[1][1]),
                        fma(-w[2], fabs(tz - tr[1][2]),
                            (v - vr[1]) + (fmin(r.l, lr[1]) + fmin(qn, qr[1])))));
                    const bool au = up >= 0.0, an = dn <= 0.0;
                    if (au) row_u[cm < kRow ? cm : kRow - 1] = (uint8_t)s;
                    cm += au ? 1 : 0;
                    if (an) row_l[cn < kRow ? cn : kRow - 1] = (uint8_t)s;
                    cn += an ? 1 : 0;
                }
                const bool finite = finite_bits(slacks);
                cm = finite ? cm : 0;
                cn = finite ? cn : 0;
                if (__ballot(cm + cn < 2 * S) == 0) {
                    // every block keeps every state: all may be the same (a constant
                    // field), and the first then stands for all.  (4096 hexahedra of 189 equal states on
                    // 24^3 nodes: 0.66 ms, 3.1 with all evaluated.)
                    const Rec3 f = L.rec[0];
                    bool differs = false;
                    for (int s = lane; s < S; s += 64) {
                        const Rec3 r = L.rec[s];
                        differs |= r.a != f.a || r.l != f.l || r.ux != f.ux || r.uy != f.uy ||
                                   r.uz != f.uz || r.nk != f.nk;
                    }
                    if (__ballot(differs) == 0) {
                        n_all = 1;
                        cm = 0;
                        cn = 0;
                    }
                }
            }

            // ---- blocks of the round in ascending order of list length: the
            // place of a block is the number of smaller (length, slot) pairs;
            // idle slots come first
            {
                int key = (cm == 0 || cm > kRow ? S : cm) + (cn == 0 || cn > kRow ? S : cn);
                if (all) key = 1;
                if (lane >= gn) key = 0;
                const unsigned mine = ((unsigned)key << 8) | (unsigned)tid;
                L.comp[tid] = mine;
                L.coord[tid] = (unsigned)(b[0] | (b[1] << 8) | (b[2] << 16));
                __syncthreads();
                int place = 0;
#pragma unroll 8
                for (int k = 0; k < kSlots; ++k) place += L.comp[k] < mine ? 1 : 0;
                // length 0: all states
                L.order[place] = (unsigned)tid | ((unsigned)(cm > kRow ? 0 : cm) << 8) |
                                 ((unsigned)(cn > kRow ? 0 : cn) << 16);
                __syncthreads();
            }
            const int first = kSlots - real;
            const int n_pass = (real + per_pass - 1) / per_pass;
            // the passes of this wave: the heaviest first, each to the wave
            // with the least work so far (every wave finds the same
            // assignment); many passes are dealt in turn
            unsigned long long mine = 0;
            const bool dealt = n_pass <= 64 && !big;
            if (dealt) {
                int last = first + (lane + 1) * per_pass - 1;
                last = last < kSlots ? last : kSlots - 1;
                const unsigned o = L.order[last];
                const int lm = (o >> 8) & 255, ln = (o >> 16) & 255;
                int work = 55 * ((lm ? lm : S) + (ln ? ln : S));
                work = (work < 67 * S ? work : 67 * S) + 900;
                int load[kWaves] = {0, 0, 0, 0};
                for (int q = n_pass - 1; q >= 0; --q) {
                    const int c = __builtin_amdgcn_readlane(work, q);
                    int w = 0, best = load[0];
#pragma unroll
                    for (int k = 1; k < kWaves; ++k)
                        if (load[k] < best) { best = load[k]; w = k; }
#pragma unroll
                    for (int k = 0; k < kWaves; ++k) load[k] += w == k ? c : 0;
                    if (w == wid) mine |= 1ull << q;
                }
            }

            // ---- evaluation
            for (int turn = 0;; ++turn) {
                int pass;
                if (dealt) {
                    if (!mine) break;
                    pass = __builtin_ctzll(mine);
                    mine &= mine - 1;
                } else {
                    if (turn * kWaves >= n_pass) break;
                    pass = turn * kWaves + wid;
                    if (pass >= n_pass && !big) break;
                }
                const int b0 = first + pass * per_pass;
                const int place = b0 + grp;
                const bool act = place < kSlots && grp < per_pass;
                const unsigned o = L.order[place < kSlots ? place : kSlots - 1];
                const int blk = o & 255;
                const int bc = L.coord[blk];
                // idle lanes take nodes of weight 0
                const int jx = act ? (bc & 255) * 2 * cg.hb[0] + 2 * px : 64;
                const int jy = ((bc >> 8) & 255) * 2 * cg.hb[1] + 2 * py;
                const int jz = (bc >> 16) * 2 * cg.hb[2] + 2 * pz;
                double x[2], y[2], z[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    x[i] = L.node[0][jx + i].u;
                    y[i] = L.node[1][jy + i].u;
                    z[i] = L.node[2][jz + i].u;
                }
                // the longest lists of the pass are those of its last block
                const unsigned last = __builtin_amdgcn_readfirstlane(
                    L.order[b0 + per_pass < kSlots ? b0 + per_pass - 1 : kSlots - 1]);
                const int lm = (last >> 8) & 255, ln = (last >> 16) & 255;
                const bool dual = big || 55 * ((lm ? lm : S) + (ln ? ln : S)) > 67 * S;
                auto values = [&](const Rec3& r, double (&v)[8]) {
                    double A[2], Y[2], Z[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const double dx = x[i] - r.ux, dy = y[i] - r.uy;
                        A[i] = fma(r.nk * dx, dx, r.a);
                        Y[i] = dy * dy;
                        Z[i] = z[i] - r.uz;
                    }
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int k = 0; k < 2; ++k) {
                            const double yz = fma(Z[k], Z[k], Y[j]);
#pragma unroll
                            for (int i = 0; i < 2; ++i) v[4 * i + 2 * j + k] = fma(r.nk, yz, A[i]);
                        }
                };
                // the envelopes of q and q_I: upper in side 0, lower in side 1
                double q[8], qi[8], ql[8], qil[8];
                if (dual) {
                    // long lists: all states, both sides at once.  Stencils
                    // beyond the staged states go chunk by chunk, staged again
                    // for every pass (all waves make the same passes then).
                    for (int c0 = 0; c0 < n_all; c0 += kCap) {
                        const int cnt = n_all - c0 < kCap ? n_all - c0 : kCap;
                        if (big) {
                            __syncthreads();
                            if (tid < cnt) {
                                Rec3 r;
                                double th;
                                (void)cull_state3(p, row0, c0 + tid, cg.inv_ns, cg.lhd, &r, &th);
                                L.rec[tid] = r;
                            }
                            __syncthreads();
                        }
                        if (c0 == 0) {
                            const Rec3 r = L.rec[0];
                            values(r, q);
#pragma unroll
                            for (int i = 0; i < 8; ++i) {
                                ql[i] = q[i];
                                qi[i] = qil[i] = q[i] + r.l;
                            }
                        }
                        for (int s = c0 == 0 ? 1 : 0; s < cnt; ++s) {
                            const Rec3 r = L.rec[s];
                            double v[8];
                            values(r, v);
#pragma unroll
                            for (int i = 0; i < 8; ++i) {
                                const double vi = v[i] + r.l;
                                q[i] = fmax(q[i], v[i]);
                                ql[i] = fmin(ql[i], v[i]);
                                qi[i] = fmax(qi[i], vi);
                                qil[i] = fmin(qil[i], vi);
                            }
                        }
                    }
                }
                // one side after the other (one code for both: fewer live
                // registers), the accumulators exchanged in between
#pragma unroll 1
                for (int side = 0; side < 2; ++side) {
                    if (!dual) {
                        // the block's list; past its end a block repeats its
                        // last state.  The lower envelope is the upper one of
                        // the negated values.
                        const double sg = side ? -1.0 : 1.0;
                        int n = (o >> (side ? 16 : 8)) & 255;
                        const uint8_t* lst = n ? L.list[side][blk] : L.all;
                        const uint8_t* const end = lst + ((n ? n : n_all) - 1);
                        n = !act ? 1 : n ? n : n_all;
                        // the index of the next state is read one step ahead
                        int i = *lst;
                        auto next = [&]() {
                            lst = lst < end ? lst + 1 : end;
                            Rec3 r = L.rec[i];
                            i = *lst;
                            r.a *= sg;
                            r.l *= sg;
                            r.nk *= sg;
                            return r;
                        };
                        {
                            const Rec3 r = next();
                            values(r, q);
#pragma unroll
                            for (int i = 0; i < 8; ++i) qi[i] = q[i] + r.l;
                        }
                        int k = 1;
                        if (__builtin_amdgcn_ballot_w64(k < n)) {
                            do {
                                const Rec3 r = next();
                                double v[8];
                                values(r, v);
#pragma unroll
                                for (int i = 0; i < 8; ++i) {
                                    const double vi = v[i] + r.l;
                                    q[i] = fmax(q[i], v[i]);
                                    qi[i] = fmax(qi[i], vi);
                                }
                                ++k;
                            } while (__builtin_amdgcn_ballot_w64(k < n));
                        }
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            q[i] *= sg;
                            qi[i] *= sg;
                        }
                    } else if (side) {
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            q[i] = ql[i];
                            qi[i] = qil[i];
                        }
                    }
                    // exps (two nodes at a time, in three phases: indices and
                    // polynomials, table reads, products) and the separable
                    // contraction M = wx wy wz over the marginals of each
                    // direction
                    double wx[2], wy[2], wz[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        wx[i] = L.node[0][jx + i].w;
                        wy[i] = L.node[1][jy + i].w;
                        wz[i] = L.node[2][jz + i].w;
                    }
                    double xt[2] = {0, 0}, yt[2] = {0, 0}, zt[2] = {0, 0}, it = 0.0;
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            ExpPrep pr[4];
                            ExpPair T[4];
#pragma unroll
                            for (int k = 0; k < 2; ++k) {
                                pr[2 * k] = exp_prep(q[4 * i + 2 * j + k]);
                                pr[2 * k + 1] = exp_prep(qi[4 * i + 2 * j + k]);
                            }
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int k = 0; k < 4; ++k) T[k] = sExp[pr[k].ni & 255];
                            __builtin_amdgcn_sched_barrier(0);
                            const double wxy = wx[i] * wy[j];
                            double t = 0.0, ti = 0.0;      // sums over z: of wz g, wz g_I
#pragma unroll
                            for (int k = 0; k < 2; ++k) {
                                const double g = exp_fin(pr[2 * k], T[2 * k]);
                                const double gi = exp_fin(pr[2 * k + 1], T[2 * k + 1]);
                                t = fma(wz[k], g, t);
                                ti = fma(wz[k], gi, ti);
                                zt[k] = fma(wxy, g, zt[k]);
                            }
                            xt[i] = fma(wy[j], t, xt[i]);
                            yt[j] = fma(wx[i], t, yt[j]);
                            it = fma(wxy, ti, it);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    const double f = side ? 1.0 - p.r_fac : 1.0 + p.r_fac;    // eq. relaxed
                    double rho = 0.0, en = 0.0, ng[3] = {0, 0, 0}, ps[3] = {0, 0, 0};
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const double mx = wx[i] * x[i], my = wy[i] * y[i], mz = wz[i] * z[i];
                        rho = fma(wx[i], xt[i], rho);
                        en = fma(mx * x[i], xt[i], en);
                        en = fma(my * y[i], yt[i], en);
                        en = fma(mz * z[i], zt[i], en);
                        ng[0] = fma(fmin(mx, 0.0), xt[i], ng[0]);
                        ps[0] = fma(fmax(mx, 0.0), xt[i], ps[0]);
                        ng[1] = fma(fmin(my, 0.0), yt[i], ng[1]);
                        ps[1] = fma(fmax(my, 0.0), yt[i], ps[1]);
                        ng[2] = fma(fmin(mz, 0.0), zt[i], ng[2]);
                        ps[2] = fma(fmax(mz, 0.0), zt[i], ps[2]);
                    }
                    // momentum (eq. mmbounds, mpbounds): the lower bound takes
                    // the upper envelope where u < 0, the lower one where
                    // u >= 0, the upper bound the reverse.  After the exchange
                    // [0] and [1] of every pair have changed places, so side 1
                    // adds to the same variables.
                    a_rho[1] = fma(f, rho, a_rho[1]);
                    a_e[1] = fma(f, fma(0.5, en, has_int * it), a_e[1]);
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        a_m[d][0] = fma(f, ng[d], a_m[d][0]);
                        a_m[d][1] = fma(f, ps[d], a_m[d][1]);
                    }
                    auto swap = [](double (&v)[2]) {
                        const double t = v[0];
                        v[0] = v[1];
                        v[1] = t;
                    };
                    swap(a_rho);
                    swap(a_e);
#pragma unroll
                    for (int d = 0; d < 3; ++d) swap(a_m[d]);
                }
            }
            __syncthreads();             // the round's lists are reused
        }

        double part[10] = {a_rho[0], a_rho[1], a_e[0], a_e[1], a_m[0][0],
                           a_m[0][1], a_m[1][0], a_m[1][1], a_m[2][0], a_m[2][1]};
        block_sum_t<kThreads, 10>(part, red);
        if (tid == 0) store_bounds<3>(p, e, part, 0);
    }
}

}  // namespace

// State indices of a row in 32 bits; grids are at most 64 nodes per direction.
bool bounds_cull_fits_3d(const BoundsArgs& a) {
    return a.nx <= 64 && a.ny <= 64 && a.nz <= 64 && a.n_s < 65536 &&
           a.nnz <= (int64_t)INT32_MAX / a.n_s;
}

hipError_t launch_bounds_cull_3d(const BoundsArgs& a, hipStream_t stream) {
    if (!bounds_cull_fits_3d(a)) return hipErrorInvalidValue;
    CullGrid3 g;
    const int n[3] = {a.nx, a.ny, a.nz};
    for (int d = 0; d < 3; ++d) {
        g.hb[d] = n[d] <= 32 ? 2 : 4;
        g.nb[d] = (n[d] + 2 * g.hb[d] - 1) / (2 * g.hb[d]);
    }
    g.inv_ns = a.n_s > 1 ? (uint32_t)(((1ull << 32) + a.n_s - 1) / a.n_s) : 0;
    g.lhd = a.half_delta > 0.0 ? log(a.half_delta) - log(2.0 * kPi) : 0.0;
    hipLaunchKernelGGL(bounds_cull_3d, dim3(bounds_grid(a)), dim3(kThreads), 0, stream, a, g);
    return hipGetLastError();
}

}  // namespace kbl
