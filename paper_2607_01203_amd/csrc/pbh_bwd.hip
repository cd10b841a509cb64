// pbh_bwd.hip -- adjoint of the path-based Hessian bound (leb_backward).
//
// Gradient of L = sum_{unit,row} g_lo r_lo + g_hi r_hi with respect to the
// nominal trajectory (z, v) and the tube (sigma, mu), for the exact-
// arithmetic bound of Theorem 1 (rounding steps are the identity; every
// selection follows the primal values and takes the first candidate in the
// order lo*lo, lo*hi, hi*lo, hi*hi on a tie).  The paper uses these
// gradients to refine the nominal point (Table II) and to penalise the
// propagated error (eq. linearization_error_cost_penalty).
//
// Interval intermediates are recomputed, never stored.  A lane owns node i of a
// timestep and spring i (to node i + 1), as in the bound kernel:
//   1. spring i primal (the bound kernel's own code): pieces of node i+1's shared
//      entries go to LDS;
//   2. node i primal and its hand-written reverse: adjoints of the node's
//      displacements, nominal attitude and thrust sum, and of the shared
//      spring pieces (the left spring's go to LDS);
//   3. spring i tangent passes: the same spring code with a forward-mode dual type
//      of two directions, five passes over the ten spring inputs (the two
//      separations; the ends of the displacements of px_i, pz_i, px_{i+1},
//      pz_{i+1}); each pass carries tangents only through what its inputs reach
//      (the displacement of pz_{i+1}, for instance, only through the fourth prefix
//      box) and contracts them with the adjoints;
//   4. per-coordinate sums in a fixed order (deterministic), then the
//      chain rule through Delta = [min(mu - sigma, 0), max(mu + sigma, 0)].
// The FP32 tangents are those of ten one-direction passes over every term, bit
// for bit: what is left out are products and sums with zero tangents.
// Rows that are unbounded, and units with invalid data, contribute nothing.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "leb.h"
#include "leb_internal.hpp"
#include "node.hpp"
#include "pbh_common.hpp"
#include "pbh_node.hpp"

namespace leb {

constexpr int BWD_MAX_U = 128;
constexpr int BWD_BLOCK = 256;           // lanes of the filled-chip form
constexpr int BWD_TASKS = 5;             // tangent passes
constexpr int BWD_SPLIT_BLOCKS = 256;    // the split form: up to one workgroup per compute unit

struct BwdArgs {
    const double* z; const double* v; const double* mu; const double* sigma;
    const double* g_lo; const double* g_hi;
    double* gz; double* gv; double* gmu; double* gsigma;
    int64_t units;
    int U, T;
    double c, kL, L0;
};

struct RowAdj { double xlo, xhi, zlo, zhi; };
struct NodeGrad { double th, s, dth[2], du1[2], du2[2], dx[2], dz[2]; };
struct PieceAdj { double lo[5], hi[5]; };
// what a lane passes to its neighbour, one after the other: spring i's pieces to
// node i+1, node i+1's piece adjoints back to spring i, spring i's gradient of
// node i+1's coordinates to node i+1
union BwdPass {
    struct { IV<float> L[5]; uint32_t unbounded; } piece;
    PieceAdj adj;
    double next[6];                      // dxn, dzn, Dxj lo/hi, Dzj lo/hi
};

// reverse of t_mul_z(a, p) for F = float (first-on-tie selections); both sides of a
// selection are added (one of them 0), so that no adjoint is addressed by a branch
__device__ __forceinline__ void bwd_mul_z(IV<float> a, IV<float> p, double tlo, double thi, double* alo,
                                          double* ahi, double* plo, double* phi) {
    const bool lf = a.lo * p.hi <= a.hi * p.lo, hf = a.lo * p.lo >= a.hi * p.hi;
    const double l1 = lf ? tlo : 0.0, l2 = lf ? 0.0 : tlo, h1 = hf ? thi : 0.0, h2 = hf ? 0.0 : thi;
    *alo += l1 * p.hi;
    *ahi += l2 * p.lo;
    *phi += l1 * a.lo;
    *plo += l2 * a.hi;
    *alo += h1 * p.lo;
    *ahi += h2 * p.hi;
    *plo += h1 * a.lo;
    *phi += h2 * a.hi;
}
// reverse of t_sq_z(a) = [0, max(a.lo^2, a.hi^2)]
__device__ __forceinline__ void bwd_sq_z(IV<float> a, double thi, double* alo, double* ahi) {
    const bool f = a.lo * a.lo >= a.hi * a.hi;
    *alo += f ? thi * 2.0 * a.lo : 0.0;
    *ahi += f ? 0.0 : thi * 2.0 * a.hi;
}

// the two tangents of pass TASK, with the spring's inputs st
template <int TASK>
__device__ __forceinline__ void bwd_task(const SpringSetup& st, double K3, double K15, double K1, double K05,
                                         AccTangent& acc) {
    auto lohi = [](IV<float> x, float ld, float le, float hd, float he) { return iv(dfm(x.lo, ld, le), dfm(x.hi, hd, he)); };
    // the displacement's own ends (lo: first tangent, hi: second)
    auto ends = [&](IV<float> x) { return lohi(x, 1.0f, 0.0f, 0.0f, 1.0f); };
    // a separation minus the displacement: its lower end moves with the displacement's upper end
    auto minus = [&](IV<float> x) { return lohi(x, 0.0f, -1.0f, -1.0f, 0.0f); };
    acc.g = acc.h = 0.0;
    if constexpr (TASK == 0)             // nominal separations dxn, dzn
        spring_core(lohi(st.dxA, 1.0f, 0.0f, 1.0f, 0.0f), lohi(st.dxB, 1.0f, 0.0f, 1.0f, 0.0f),
                    lohi(st.dz0, 0.0f, 1.0f, 0.0f, 1.0f), lohi(st.dz1, 0.0f, 1.0f, 0.0f, 1.0f),
                    lohi(st.dz2, 0.0f, 1.0f, 0.0f, 1.0f), st.Dxi, st.Dzi, st.Dxj, st.Dzj, 1.0, 1.0, 1.0, 1.0, K3, K15,
                    K1, K05, acc, acc);
    else if constexpr (TASK == 1)        // Dxi
        spring_core(minus(st.dxA), minus(st.dxB), st.dz0, st.dz1, st.dz2, ends(st.Dxi), st.Dzi, st.Dxj, st.Dzj, 1.0, 1.0,
                    1.0, 1.0, K3, K15, K1, K05, acc, acc);
    else if constexpr (TASK == 2)        // Dzi
        spring_core(st.dxA, st.dxB, st.dz0, minus(st.dz1), minus(st.dz2), st.Dxi, ends(st.Dzi), st.Dxj, st.Dzj, 1.0, 1.0,
                    1.0, 1.0, K3, K15, K1, K05, acc, acc);
    else if constexpr (TASK == 3)        // Dxj
        spring_core(st.dxA, ends(st.dxB), st.dz0, st.dz1, st.dz2, st.Dxi, st.Dzi, ends(st.Dxj), st.Dzj, 1.0, 1.0, 1.0, 1.0,
                    K3, K15, K1, K05, acc, acc);
    else                                 // Dzj
        spring_core(st.dxA, st.dxB, st.dz0, st.dz1, ends(st.dz2), st.Dxi, st.Dzi, st.Dxj, ends(st.Dzj), 1.0, 1.0, 1.0,
                    1.0, K3, K15, K1, K05, acc, acc);
}

// The adjoint of the timesteps of one workgroup: lane ln of `copy` holds node i of
// timestep lt (its inputs d, the adjoints of its own and the next node's rows).  Contains
// four workgroup barriers; returns whether this lane holds a node's result.
template <bool SPLIT> struct BwdShared {
    static constexpr int LANES = SPLIT ? 64 : BWD_BLOCK, COPIES = SPLIT ? BWD_TASKS : 1;
    BwdPass pass[COPIES][LANES];
    uint32_t unb[COPIES][LANES];                               // row unbounded
    uint32_t flag[COPIES][LANES];                              // per timestep
    double grad[SPLIT ? LANES : 1][2 * BWD_TASKS];
};
struct BwdConsts { int U; double c, kL, L0; };
struct BwdOut { double nom[8], mu[8], sigma[8]; };             // per coordinate of the node

template <bool SPLIT>
__device__ __forceinline__ bool bwd_core(const BwdConsts& K, BwdShared<SPLIT>& H, const NodeIn& d, RowAdj gi, RowAdj gj,
                                         int wave, int copy, int ln, int lt, int i, bool active, bool right,
                                         BwdOut& out) {
    const int U = K.U;
    const IV<float> Dx = disp_interval(d.ms[0], d.ss[0]), Dz = disp_interval(d.ms[1], d.ss[1]);
    __syncthreads();
    if (active && (node_flags(d) & LEB_FLAG_BAD_INPUT)) atomicOr(&H.flag[copy][lt], LEB_FLAG_BAD_INPUT);
    const double K3 = 3.0 * K.kL * K.c, K15 = 1.5 * K.kL * K.c, K1 = K.kL * K.c, K05 = 0.5 * K.kL * K.c;

    // ---- 1. spring i primal
    IV<float> R[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) R[q] = iv(0.0f, 0.0f);
    bool spring_ok = false;
    SpringSetup st;
    if (right) {
        spring_setup_v(d.zs[0], d.zs[1], d.zj[0], d.zj[1], Dx, Dz, disp_interval(d.mj[0], d.sj[0]),
                       disp_interval(d.mj[1], d.sj[1]), K.L0, st);
        AccPrimal acc;
        SpringPieces pc;
        spring_ok = spring_core(st.dxA, st.dxB, st.dz0, st.dz1, st.dz2, st.Dxi, st.Dzi, st.Dxj, st.Dzj, 1.0, 1.0, 1.0,
                                1.0, K3, K15, K1, K05, acc, pc);
        BwdPass& o = H.pass[copy][ln];
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            o.piece.L[q] = spring_ok ? pc.L[q] : iv(0.0f, 0.0f);
            R[q] = spring_ok ? pc.R[q] : iv(0.0f, 0.0f);
        }
        o.piece.unbounded = spring_ok ? 0u : 1u;
    }
    __syncthreads();

    // ---- 2. node i primal + reverse
    const bool bad = active && (H.flag[copy][lt] & LEB_FLAG_BAD_INPUT);
    uint32_t row_unb = (right && !spring_ok) ? 1u : 0u;
    PieceAdj rbar;
#pragma unroll
    for (int q = 0; q < 5; ++q) { rbar.lo[q] = 0.0; rbar.hi[q] = 0.0; }
    NodeGrad ng = {};
    if (active) {
        IV<float> L[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) L[q] = iv(0.0f, 0.0f);
        if (i > 0) {
            const BwdPass& o = H.pass[copy][ln - 1];
            row_unb |= o.piece.unbounded;
#pragma unroll
            for (int q = 0; q < 5; ++q) L[q] = o.piece.L[q];
        }
        H.unb[copy][ln] = row_unb;
        RowAdj g = gi;
        if (row_unb || bad) { g.xlo = g.xhi = g.zlo = g.zhi = 0.0; }
        const bool own = U > 1 && !row_unb;
        NodeTerms nt;
        const IV<float> Dth = disp_interval(d.ms[2], d.ss[2]), Du1 = disp_interval(d.ms[6], d.ss[6]),
                        Du2 = disp_interval(d.ms[7], d.ss[7]);
        const double thn = d.zs[2], sn = d.vs[0] + d.vs[1];
        node_terms(thn, sn, Dth, Du1, Du2, Dx, Dz, R, L, own, K.c, K15, K1, K05, 1.0, 1.0, 1.0, 1.0, 1.0, nt);
        // term adjoints
        double tlo[12], thi[12];
        double sbar = 0.0;
#pragma unroll
        for (int q = 0; q < 12; ++q) {
            const int row = node_term_row(q);
            const double alo = row == 0 ? g.xlo : g.zlo, ahi = row == 0 ? g.xhi : g.zhi;
            const double k = nt.k[q];
            tlo[q] = k * (nt.neg[q] ? ahi : alo);
            thi[q] = k * (nt.neg[q] ? alo : ahi);
            if (q == 0 || q == 3) {
                // d kappa / d s~ = +-c/2 ; kappa enters through the selected endpoints
                const float a = nt.neg[q] ? nt.T[q].hi : nt.T[q].lo;
                const float b = nt.neg[q] ? nt.T[q].lo : nt.T[q].hi;
                const double dk = (q == 0 ? 0.5 : -0.5) * K.c;
                sbar += dk * (alo * (double)a + ahi * (double)b);
            }
        }
        ng.s = sbar;
        double Sb_lo = 0, Sb_hi = 0, Cb_lo = 0, Cb_hi = 0;
        double Ptt_lo = 0, Ptt_hi = 0, Pu1_lo = 0, Pu1_hi = 0, Pu2_lo = 0, Pu2_hi = 0;
        const IV<float> S = iv(nt.sc.s.lo, nt.sc.s.hi), Cs = iv(nt.sc.c.lo, nt.sc.c.hi);
        bwd_mul_z(S, nt.Ptt, tlo[0], thi[0], &Sb_lo, &Sb_hi, &Ptt_lo, &Ptt_hi);
        bwd_mul_z(Cs, nt.Ptu1, tlo[1], thi[1], &Cb_lo, &Cb_hi, &Pu1_lo, &Pu1_hi);
        bwd_mul_z(Cs, nt.Ptu2, tlo[2], thi[2], &Cb_lo, &Cb_hi, &Pu2_lo, &Pu2_hi);
        bwd_mul_z(Cs, nt.Ptt, tlo[3], thi[3], &Cb_lo, &Cb_hi, &Ptt_lo, &Ptt_hi);
        bwd_mul_z(S, nt.Ptu1, tlo[4], thi[4], &Sb_lo, &Sb_hi, &Pu1_lo, &Pu1_hi);
        bwd_mul_z(S, nt.Ptu2, tlo[5], thi[5], &Sb_lo, &Sb_hi, &Pu2_lo, &Pu2_hi);
        // displacement products of the attitude block
        bwd_sq_z(Dth, Ptt_hi, &ng.dth[0], &ng.dth[1]);
        bwd_mul_z(Dth, Du1, Pu1_lo, Pu1_hi, &ng.dth[0], &ng.dth[1], &ng.du1[0], &ng.du1[1]);
        bwd_mul_z(Dth, Du2, Pu2_lo, Pu2_hi, &ng.dth[0], &ng.dth[1], &ng.du2[0], &ng.du2[1]);
        // sin / cos bounds -> Theta endpoints -> nominal theta and Dth
        const double a64 = thn + (double)Dth.lo, b64 = thn + (double)Dth.hi;
        double Th_lo = 0.0, Th_hi = 0.0;
        {
            const SinCos& sc = nt.sc;
            // sine and cosine at both ends; the derivative of an end's selected value, 0
            // when the bound is a clamped extremum (selection 2)
            double sa, ca, sb, cb;
            if (sc.wide) {
                sincos(a64, &sa, &ca);
                sincos(b64, &sb, &cb);
            } else {
                sa = (double)sin_poly(sc.fa); ca = (double)cos_poly(sc.fa);
                sb = (double)sin_poly(sc.fb); cb = (double)cos_poly(sc.fb);
            }
            const double dslo = sc.s_lo == 0 ? ca : cb, dshi = sc.s_hi == 0 ? ca : cb;
            const double dclo = sc.c_lo == 0 ? -sa : -sb, dchi = sc.c_hi == 0 ? -sa : -sb;
            auto ends = [&](int sel, double x) {
                Th_lo += sel == 0 ? x : 0.0;
                Th_hi += sel == 1 ? x : 0.0;
            };
            ends(sc.s_lo, Sb_lo * dslo);
            ends(sc.s_hi, Sb_hi * dshi);
            ends(sc.c_lo, Cb_lo * dclo);
            ends(sc.c_hi, Cb_hi * dchi);
        }
        ng.th = Th_lo + Th_hi;
        ng.dth[0] += Th_lo;
        ng.dth[1] += Th_hi;
        // own position pairs
        PieceAdj lbar;
#pragma unroll
        for (int q = 0; q < 5; ++q) { lbar.lo[q] = 0.0; lbar.hi[q] = 0.0; }
        if (own) {
            double Gb_lo[5] = {0, 0, 0, 0, 0}, Gb_hi[5] = {0, 0, 0, 0, 0};
            double Pxx_lo = 0, Pxx_hi = 0, Pxz_lo = 0, Pxz_hi = 0, Pzz_lo = 0, Pzz_hi = 0;
            bwd_mul_z(nt.G[0], nt.Pxx, tlo[6], thi[6], &Gb_lo[0], &Gb_hi[0], &Pxx_lo, &Pxx_hi);
            bwd_mul_z(nt.G[1], nt.Pxz, tlo[7], thi[7], &Gb_lo[1], &Gb_hi[1], &Pxz_lo, &Pxz_hi);
            bwd_mul_z(nt.G[3], nt.Pzz, tlo[8], thi[8], &Gb_lo[3], &Gb_hi[3], &Pzz_lo, &Pzz_hi);
            bwd_mul_z(nt.G[1], nt.Pxx, tlo[9], thi[9], &Gb_lo[1], &Gb_hi[1], &Pxx_lo, &Pxx_hi);
            bwd_mul_z(nt.G[2], nt.Pxz, tlo[10], thi[10], &Gb_lo[2], &Gb_hi[2], &Pxz_lo, &Pxz_hi);
            bwd_mul_z(nt.G[4], nt.Pzz, tlo[11], thi[11], &Gb_lo[4], &Gb_hi[4], &Pzz_lo, &Pzz_hi);
            bwd_sq_z(Dx, Pxx_hi, &ng.dx[0], &ng.dx[1]);
            bwd_mul_z(Dx, Dz, Pxz_lo, Pxz_hi, &ng.dx[0], &ng.dx[1], &ng.dz[0], &ng.dz[1]);
            bwd_sq_z(Dz, Pzz_hi, &ng.dz[0], &ng.dz[1]);
            // G = R - L: [R.lo - L.hi, R.hi - L.lo]
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                rbar.lo[q] = Gb_lo[q]; rbar.hi[q] = Gb_hi[q];
                lbar.hi[q] = -Gb_lo[q]; lbar.lo[q] = -Gb_hi[q];
            }
        }
        if (i > 0) H.pass[copy][ln - 1].adj = lbar;
    }
    __syncthreads();

    // ---- 3. spring i tangent passes
    double sg[2 * BWD_TASKS];            // dxn, dzn, Dxi lo/hi, Dzi lo/hi, Dxj lo/hi, Dzj lo/hi
#pragma unroll
    for (int q = 0; q < 2 * BWD_TASKS; ++q) sg[q] = 0.0;
    if (right && spring_ok) {
        const PieceAdj lb = H.pass[copy][ln].adj;
        if (bad || row_unb) gi = RowAdj{0.0, 0.0, 0.0, 0.0};
        if (bad || H.unb[copy][ln + 1]) gj = RowAdj{0.0, 0.0, 0.0, 0.0};
        AccTangent acc;
        // slot adjoints: row i takes C + B, row i+1 takes -(C + A)
        acc.alo[S_CX] = gi.xlo - gj.xhi; acc.ahi[S_CX] = gi.xhi - gj.xlo;
        acc.alo[S_CZ] = gi.zlo - gj.zhi; acc.ahi[S_CZ] = gi.zhi - gj.zlo;
        acc.alo[S_BX] = gi.xlo;          acc.ahi[S_BX] = gi.xhi;
        acc.alo[S_BZ] = gi.zlo;          acc.ahi[S_BZ] = gi.zhi;
        acc.alo[S_AX] = -gj.xhi;         acc.ahi[S_AX] = -gj.xlo;
        acc.alo[S_AZ] = -gj.zhi;         acc.ahi[S_AZ] = -gj.zlo;
        acc.rlo = rbar.lo; acc.rhi = rbar.hi; acc.llo = lb.lo; acc.lhi = lb.hi;
        auto run = [&](auto task) {
            constexpr int Q = decltype(task)::value;
            if (SPLIT && wave != Q) return;
            bwd_task<Q>(st, K3, K15, K1, K05, acc);
            if (SPLIT) { H.grad[ln][2 * Q] = acc.g; H.grad[ln][2 * Q + 1] = acc.h; }
            else { sg[2 * Q] = acc.g; sg[2 * Q + 1] = acc.h; }
        };
        run(std::integral_constant<int, 0>()); run(std::integral_constant<int, 1>());
        run(std::integral_constant<int, 2>()); run(std::integral_constant<int, 3>());
        run(std::integral_constant<int, 4>());
    } else if (SPLIT && active) {
        H.grad[ln][2 * wave] = 0.0;
        H.grad[ln][2 * wave + 1] = 0.0;
    }
    if (SPLIT) {
        __syncthreads();
        if (wave > 0) return false;      // the first wave adds up
        if (active) {
#pragma unroll
            for (int q = 0; q < 2 * BWD_TASKS; ++q) sg[q] = H.grad[ln][q];
        }
    } else {
        if (right) {
            double* o = H.pass[0][ln].next;
            o[0] = sg[0]; o[1] = sg[1];
#pragma unroll
            for (int q = 0; q < 4; ++q) o[2 + q] = sg[6 + q];
        }
        __syncthreads();
    }
    if (!active) return false;

    // ---- 4. per-coordinate sums (fixed order) and the box chain rule
    double lf[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};             // spring i-1: node i is its second node
    if (i > 0) {
#pragma unroll
        for (int q = 0; q < 6; ++q)
            lf[q] = SPLIT ? H.grad[ln - 1][q < 2 ? q : q + 4] : H.pass[0][ln - 1].next[q];
    }
    const double gn[8] = {lf[0] - sg[0], lf[1] - sg[1], ng.th, 0.0, 0.0, 0.0, ng.s, ng.s};
    const double gl[8] = {ng.dx[0] + sg[2] + lf[2], ng.dz[0] + sg[4] + lf[4], ng.dth[0], 0.0, 0.0, 0.0, ng.du1[0],
                           ng.du2[0]};
    const double gh[8] = {ng.dx[1] + sg[3] + lf[3], ng.dz[1] + sg[5] + lf[5], ng.dth[1], 0.0, 0.0, 0.0, ng.du1[1],
                           ng.du2[1]};
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const double sgm = d.ss[c], mu = d.ms[c];
        // Delta_lo = min(mu - sigma, 0), Delta_hi = max(mu + sigma, 0); first candidate on a tie
        const double alo = !bad && (mu - sgm <= 0.0) ? gl[c] : 0.0;
        const double ahi = !bad && (mu + sgm >= 0.0) ? gh[c] : 0.0;
        out.sigma[c] = ahi - alo;
        out.mu[c] = alo + ahi;
        out.nom[c] = bad ? 0.0 : gn[c];
    }
    return true;
}

// SPLIT = false: 256 lanes, each runs its spring's five passes one after the other.
// SPLIT = true (launches that leave the chip idle): five waves over the same up
// to 64 lanes, each wave runs phases 1 and 2 for itself and then one pass.
//
// What bounds it: VALU issue (10,500 instructions a wave, most of them in phase
// 3) at two waves a SIMD when the chip is full (256 registers, 24 of them spilled), the
// serial chain of one lane otherwise.  28 nodes, 256 x 40 steps: 102 us (337 us with ten one-direction passes
// over every term, whose hoisted values took 430 registers, one wave a SIMD, and
// with adjoints addressed through scratch); 1 x 40: 15 us (55 us).
template <bool SPLIT>
__global__ void __launch_bounds__(SPLIT ? 64 * BWD_TASKS : BWD_BLOCK, SPLIT ? 1 : 2) pbh_chain_bwd(BwdArgs A) {
    __shared__ BwdShared<SPLIT> S;
    const int U = A.U, T = A.T, nx = 6 * U, nu = 2 * U, n = nx + nu;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int copy = SPLIT ? wave : 0, ln = SPLIT ? (threadIdx.x & 63) : threadIdx.x;
    const int64_t u0 = (int64_t)blockIdx.x * T;
    const int64_t left = A.units - u0;
    const int nloc = left < T ? (int)left : T;
    const int lt = ln / U, i = ln - lt * U;
    const bool active = lt < nloc, right = active && i < U - 1;
    S.flag[copy][ln] = 0u;
    TileRef tr = {};
    tr.Z = A.z + u0 * nx; tr.V = A.v + u0 * nu; tr.MU = A.mu ? A.mu + u0 * n : nullptr; tr.SG = A.sigma + u0 * n;
    tr.nloc = nloc;
    NodeIn d;
    node_load(tr, U, lt, i, d);
    RowAdj gi = {0.0, 0.0, 0.0, 0.0}, gj = {0.0, 0.0, 0.0, 0.0};
    if (active) {
        const double* gl = A.g_lo + (u0 + lt) * nx + 6 * i;
        const double* gh = A.g_hi + (u0 + lt) * nx + 6 * i;
        gi = RowAdj{gl[3], gh[3], gl[4], gh[4]};
        if (right) gj = RowAdj{gl[9], gh[9], gl[10], gh[10]};
    }
    BwdOut o;
    const BwdConsts K{U, A.c, A.kL, A.L0};
    if (!bwd_core<SPLIT>(K, S, d, gi, gj, wave, copy, ln, lt, i, active, right, o)) return;
    const int64_t u = u0 + lt;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const int64_t q = u * n + (c < 6 ? 6 * i + c : nx + 2 * i + c - 6);
        A.gsigma[q] = o.sigma[c];
        if (A.gmu) A.gmu[q] = o.mu[c];
        if (c < 6) A.gz[u * nx + 6 * i + c] = o.nom[c];
        else A.gv[u * nu + 2 * i + c - 6] = o.nom[c];
    }
}

// The whole descent on the nominal point (pgd.hip) of up to 64 / U timesteps in one
// workgroup: timesteps are independent of each other, so nothing leaves it between the
// steps.  Waves 0 .. 4: the adjoint (upstream -1 on the lower, +1 on the upper ends), the
// first also the move; wave 5: the bound at the same iterate, for its width.
//
// What bounds it: the serial chain of the adjoint, 19 us an iteration (256 registers, 25
// spilled).  28 nodes, 40 timesteps, 10 steps: 209 us (a launch each for the bound, the
// adjoint and the move: 300 us).
constexpr int PGD_WAVES = BWD_TASKS + 1;

struct PgdChainArgs {
    const double* z0; const double* v0; const double* mu0; const double* sigma;
    double* zo; double* vo; double* width; double* width0;
    int64_t units;
    int U, T, steps, fixed_box;
    double radius, lr;
    double c, kL, L0, pad;
    int compact;
};

__global__ void __launch_bounds__(64 * PGD_WAVES, 1) pgd_chain_kernel(PgdChainArgs A) {
    __shared__ BwdShared<true> S;
    // the iterate and its mu, sigma, the start, mu0, the best iterate; the bound's rows
    __shared__ __attribute__((aligned(16))) double sz[64 * 6], sv[64 * 2], smu[64 * 8], ssg[64 * 8], sz0[64 * 6],
        sv0[64 * 2], smu0[64 * 8], szb[64 * 6], svb[64 * 2], rlo[64 * 6], rhi[64 * 6], sg[64 * 8];
    __shared__ uint32_t s_better[64];
    __shared__ SpringOut s_sp[64];
    __shared__ uint32_t s_fl[64];
    const int U = A.U, T = A.T, nx = 6 * U, nu = 2 * U, n = nx + nu, tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), ln = tid & 63;
    const int64_t u0 = (int64_t)blockIdx.x * T, rest = A.units - u0;
    const int nloc = rest < T ? (int)rest : T;
    for (int q = tid; q < nloc * nx; q += 64 * PGD_WAVES) sz[q] = sz0[q] = szb[q] = A.z0[u0 * nx + q];
    for (int q = tid; q < nloc * nu; q += 64 * PGD_WAVES) sv[q] = sv0[q] = svb[q] = A.v0[u0 * nu + q];
    for (int q = tid; q < nloc * n; q += 64 * PGD_WAVES) {
        smu[q] = smu0[q] = A.mu0 ? A.mu0[u0 * n + q] : 0.0;
        ssg[q] = A.sigma[u0 * n + q];
    }
    double best = INFINITY;
    const TileRef t0{sz, sv, smu, ssg, rlo, rhi, nullptr, nullptr, nullptr, nloc};
    for (int st = 0; st <= A.steps; ++st) {
        // (the lane's place is formed anew each time, or the addresses of everything it
        // reads would be kept in registers over the loop)
        int lp = ln, Up = U;
        asm volatile("" : "+v"(lp), "+s"(Up));
        const int lt = lp / Up, i = lp - lt * Up;
        const bool active = lt < nloc, right = active && i < U - 1;
        const RowAdj gi = active ? RowAdj{-1.0, 1.0, -1.0, 1.0} : RowAdj{0.0, 0.0, 0.0, 0.0};
        const RowAdj gj = right ? RowAdj{-1.0, 1.0, -1.0, 1.0} : RowAdj{0.0, 0.0, 0.0, 0.0};
        double c_ = A.c, kL_ = A.kL, L0_ = A.L0;
        asm volatile("" : "+s"(c_), "+s"(kL_), "+s"(L0_));
        const BwdConsts K{U, c_, kL_, L0_};
        if (wave < BWD_TASKS) S.flag[wave][ln] = 0u;
        else s_fl[ln] = 0u;
        __syncthreads();                             // the iterate is written
        if (wave == BWD_TASKS) {
            NodeIn d;
            node_load(t0, U, lt, i, d);
            wave_lds_fence();                        // s_fl cleared
            node_pass<true>(A, t0, d, lt, i, s_sp, s_fl);
            if (st < A.steps) {                      // the barriers of bwd_core
                __syncthreads();
                __syncthreads();
                __syncthreads();
            }
            __syncthreads();
        } else if (st < A.steps) {
            NodeIn d;
            node_load(t0, U, lt, i, d);
            BwdOut o;
            if (bwd_core<true>(K, S, d, gi, gj, wave, wave, ln, lt, i, active, right, o)) {
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    sg[lt * n + (c < 6 ? 6 * i + c : nx + 2 * i + c - 6)] = A.fixed_box ? o.nom[c] - o.mu[c] : o.nom[c];
                }
            }
        } else {
            __syncthreads();
        }
        if (wave == 0) {
            // the vx and vz rows' widths, summed in row order by the timestep's first lane
            double w = 0.0;
            if (active && i == 0) {
                const double* lo = rlo + lt * nx;
                const double* hi = rhi + lt * nx;
                for (int q = 0; q < U; q += 4) {
                    double x[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int nd = q + (e >> 1) < U ? q + (e >> 1) : 0;
                        x[e] = hi[6 * nd + 3 + (e & 1)] - lo[6 * nd + 3 + (e & 1)];
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (q + (e >> 1) < U) w += x[e];
                }
            }
            if (active && i == 0) {
                const bool better = w < best;
                if (st == 0 && A.width0) A.width0[u0 + lt] = w;
                if (better) best = w;
                s_better[lt] = better ? 1u : 0u;
            }
            wave_lds_fence();
            const double frac = st < A.steps ? A.lr * (1.0 - (double)st / A.steps) : 0.0;
            for (int q = ln; q < nloc * n; q += 64) {
                const int l = q / n, c = q - l * n;
                double* ap = c < nx ? sz + l * nx + c : sv + l * nu + c - nx;
                const double a0 = *(c < nx ? sz0 + l * nx + c : sv0 + l * nu + c - nx);
                double x = *ap;
                if (s_better[l]) *(c < nx ? szb + l * nx + c : svb + l * nu + c - nx) = x;
                if (st == A.steps) continue;
                const double g = sg[q], r = A.radius * ssg[q];
                if (g > 0.0) x -= frac * r;
                else if (g < 0.0) x += frac * r;
                x = fmin(fmax(x, a0 - r), a0 + r);
                *ap = x;
                if (A.fixed_box) smu[q] = a0 + (A.mu0 ? smu0[q] : 0.0) - x;
            }
        }
    }
    __syncthreads();
    for (int q = tid; q < nloc * nx; q += 64 * PGD_WAVES) A.zo[u0 * nx + q] = szb[q];
    for (int q = tid; q < nloc * nu; q += 64 * PGD_WAVES) A.vo[u0 * nu + q] = svb[q];
    if (wave == 0 && ln < nloc * U && ln % U == 0) A.width[u0 + ln / U] = best;
}

int launch_pbh_bwd(const leb_dynamics* dyn, int64_t units, const double* z, const double* v, const double* mu,
                   const double* sigma, const double* g_lo, const double* g_hi, double* gz, double* gv,
                   double* gmu, double* gsigma, hipStream_t stream) {
    if (dyn->n_units > BWD_MAX_U) return LEB_ENOTSUP;
    BwdArgs a;
    a.z = z; a.v = v; a.mu = mu; a.sigma = sigma; a.g_lo = g_lo; a.g_hi = g_hi;
    a.gz = gz; a.gv = gv; a.gmu = gmu; a.gsigma = gsigma;
    a.units = units;
    a.U = dyn->n_units;
    a.c = dyn->dt / dyn->m;
    a.kL = dyn->k_spring * dyn->rest_len;
    a.L0 = dyn->rest_len;
    // the split form while every workgroup has a compute unit of its own (28 nodes, whole
    // call: 320 units 16.7 us, unsplit 26.0; 640 units 29.8 and 26.6); chains of more than 64
    // nodes do not fit its lanes
    const int ts = a.U <= 64 ? 64 / a.U : 0;
    const bool split = ts > 0 && (units + ts - 1) / ts <= BWD_SPLIT_BLOCKS;
    a.T = split ? ts : BWD_BLOCK / a.U;
    const int64_t blocks = (units + a.T - 1) / a.T;
    if (blocks > 0x7fffffff) return LEB_EINVAL;
    if (split) hipLaunchKernelGGL(pbh_chain_bwd<true>, dim3((unsigned)blocks), dim3(64 * BWD_TASKS), 0, stream, a);
    else hipLaunchKernelGGL(pbh_chain_bwd<false>, dim3((unsigned)blocks), dim3(BWD_BLOCK), 0, stream, a);
    return hipGetLastError() == hipSuccess ? LEB_OK : LEB_EDEVICE;
}

// The fused descent while every workgroup has a compute unit of its own (28 nodes, 10 steps,
// whole call: 40 timesteps 211 us and 309 by launches, 480 timesteps 218 and 320; from
// then on the workgroups would take turns) and the launch stays below 0.1 s (19 us a step: a
// longer one would hold the device, and could not be ended); *done = false: not that case,
// nothing launched.
constexpr int PGD_FUSED_STEPS = 4096;

int launch_pgd_chain(const leb_dynamics* dyn, int64_t units, const double* z0, const double* v0, const double* mu0,
                     const double* sigma, int fixed_box, double radius, int steps, double lr, double* z, double* v,
                     double* width, double* width0, hipStream_t stream, bool* done) {
    const int U = dyn->n_units, T = U <= 64 ? 64 / U : 0;
    *done = T > 0 && (units + T - 1) / T <= BWD_SPLIT_BLOCKS && steps <= PGD_FUSED_STEPS;
    if (!*done) return LEB_OK;
    PgdChainArgs a;
    a.z0 = z0; a.v0 = v0; a.mu0 = mu0; a.sigma = sigma;
    a.zo = z; a.vo = v; a.width = width; a.width0 = width0;
    a.units = units;
    a.U = U; a.T = T; a.steps = steps; a.fixed_box = fixed_box;
    a.radius = radius; a.lr = lr;
    a.c = dyn->dt / dyn->m;
    a.kL = dyn->k_spring * dyn->rest_len;
    a.L0 = dyn->rest_len;
    a.pad = 0.0; a.compact = 0;
    hipLaunchKernelGGL(pgd_chain_kernel, dim3((unsigned)((units + T - 1) / T)), dim3(64 * PGD_WAVES), 0, stream, a);
    return hipGetLastError() == hipSuccess ? LEB_OK : LEB_EDEVICE;
}

}  // namespace leb

using namespace leb;

extern "C" int leb_backward(const leb_dynamics* dyn, int32_t batch, int32_t N, const double* z, const double* v,
                            const double* mu, const double* sigma, const double* g_lo, const double* g_hi,
                            double* gz, double* gv, double* gmu, double* gsigma, void* stream) {
    int rc = check_chain_dynamics(dyn);
    if (rc != LEB_OK) return rc;
    if (dyn->kind != LEB_DYN_PQUAD_CHAIN) return LEB_ENOTSUP;
    if (batch < 0 || N < 0) return LEB_EINVAL;
    if (gmu && !mu) return LEB_EINVAL;
    const int64_t units = (int64_t)batch * N;
    if (units == 0) return LEB_OK;
    if (!z || !v || !sigma || !g_lo || !g_hi || !gz || !gv || !gsigma) return LEB_EINVAL;
    const void* ptrs[] = {z, v, mu, sigma, g_lo, g_hi, gz, gv, gmu, gsigma};
    for (const void* p : ptrs)
        if (p && !aligned8(p)) return LEB_EINVAL;
    return launch_pbh_bwd(dyn, units, z, v, mu, sigma, g_lo, g_hi, gz, gv, gmu, gsigma, (hipStream_t)stream);
}
