// pbh_node.hpp -- one node of one timestep of the chain in the path-based
// Hessian bound (Theorem 1): its coordinates loaded into registers, spring
// i (to node i+1) and the node's two non-linear rows.  Shared by the bound
// kernel and the fused fixed-point sweep, so both evaluate the same
// expressions in the same order.
//
// A lane holds node i of timestep t.  spring_step evaluates spring i and
// hands node i+1 its terms (a SpringOut in LDS); after a barrier that
// covers the lanes of the timestep, node_step adds the left spring's terms
// and the attitude block and returns the node's rows 3 (vx) and 4 (vz).
#pragma once
#include "ivl.hpp"
#include "node.hpp"
#include "pbh_common.hpp"

namespace leb {

struct SpringOut {      // what spring i passes to node i+1 (row i+1)
    double xlo, xhi, zlo, zhi;      // -(cross + own-of-node-i terms), already scaled
    IV<float> L[5];                 // node i+1's shared own-position entries
    uint32_t unbounded;
    uint32_t pad_;
};

// T timesteps with their own pointers (nloc <= T of them present).
struct TileRef {
    const double *Z, *V, *MU, *SG;
    double *RLO, *RHI, *CB, *RB;
    uint32_t* FL;
    int nloc;
};

// A pointer known to address global memory (loads and stores through it need not be
// flat, which would tie their waits to those of LDS).
template <class T> __device__ __forceinline__ T* global_ptr(T* p) {
    return (T*)(__attribute__((address_space(1))) T*)p;
}

typedef double node_d2 __attribute__((ext_vector_type(2), aligned(8)));

// Coordinates of node i at one timestep (state rows 6i.., inputs 2i..) and
// the positions of node i+1 that spring i needs.
struct NodeIn { double zs[6], vs[2], ms[8], ss[8], zj[2], mj[2], sj[2]; };

// Every load is unconditional, two doubles at a time, from a clamped place: a lane
// past the last timestep reads the first one's, the last node its own position again.
__device__ __forceinline__ void node_load(const TileRef& t, int U, int lt, int i, NodeIn& d) {
    const int nx = 6 * U, nu = 2 * U, n = nx + nu;
    const bool active = lt < t.nloc;
    const int l = active ? lt : 0, c = active ? i : 0, cj = c < U - 1 ? c + 1 : c;
    const double* zp = t.Z + (int64_t)l * nx;
    const double* vp = t.V + (int64_t)l * nu;
    const double* sp = t.SG + (int64_t)l * n;
    auto pair = [](const double* p, double* o) {
        const node_d2 x = *reinterpret_cast<const node_d2*>(p);
        o[0] = x[0];
        o[1] = x[1];
    };
#pragma unroll
    for (int q = 0; q < 6; q += 2) { pair(zp + 6 * c + q, d.zs + q); pair(sp + 6 * c + q, d.ss + q); }
    pair(vp + 2 * c, d.vs);
    pair(sp + nx + 2 * c, d.ss + 6);
    pair(zp + 6 * cj, d.zj);
    pair(sp + 6 * cj, d.sj);
    if (t.MU) {
        const double* mp = t.MU + (int64_t)l * n;
#pragma unroll
        for (int q = 0; q < 6; q += 2) pair(mp + 6 * c + q, d.ms + q);
        pair(mp + nx + 2 * c, d.ms + 6);
        pair(mp + 6 * cj, d.mj);
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) d.ms[q] = 0.0;
        d.mj[0] = d.mj[1] = 0.0;
    }
}

// input flags of the node's coordinates (bad input, hull extended)
__device__ __forceinline__ uint32_t node_flags(const NodeIn& d) {
    uint32_t f = 0;
#pragma unroll
    for (int c = 0; c < 6; ++c)
        if (!isfinite(d.zs[c])) f |= LEB_FLAG_BAD_INPUT;
    if (!isfinite(d.vs[0]) || !isfinite(d.vs[1])) f |= LEB_FLAG_BAD_INPUT;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        if (!isfinite(d.ss[c]) || !isfinite(d.ms[c]) || !(d.ss[c] >= 0.0)) f |= LEB_FLAG_BAD_INPUT;
        if (fabs(d.ms[c]) > d.ss[c]) f |= LEB_FLAG_HULL_EXTENDED;
    }
    return f;
}

struct NodeConsts {
    double c;        // dt / m
    double L0;       // spring rest length
    double K3, K15, K1, K05;   // 3, 1.5, 1, 0.5 times k_spring rest_len c (all >= 0 for k_spring >= 0)
};
__device__ __forceinline__ NodeConsts node_consts(double c, double kL, double L0) {
    NodeConsts k;
    k.c = c; k.L0 = L0;
    k.K3 = 3.0 * kL * c; k.K15 = 1.5 * kL * c; k.K1 = kL * c; k.K05 = 0.5 * kL * c;
    return k;
}

// what a lane keeps from spring_step for node_step
struct SpringKeep {
    IV<float> Dx, Dz, Dth, Du1, Du2;
    div_ rx, rz;          // spring i's terms for row i
    IV<float> R[5];       // node i's shared own-position entries (right spring)
    uint32_t unb;         // spring i has no finite bound
};

// Spring i (nodes i, i+1); writes *out and returns whether the spring is unbounded through
// k.unb.  Every lane evaluates it (the last node of a chain against itself) and a lane
// without a spring drops the result: branches around it cost more in register moves
// than they save (28 nodes, 2,560 x 40, whole call: 135 us, with the branches 141; where
// every spring is unbounded the branches would save 0.5 us of a launch).  springs: the
// chain has any.
__device__ __forceinline__ void spring_step(const NodeConsts& K, const NodeIn& d, bool springs, bool right, SpringKeep& k,
                                            SpringOut* out) {
    k.Dx = disp_interval(d.ms[0], d.ss[0]); k.Dz = disp_interval(d.ms[1], d.ss[1]);
    k.Dth = disp_interval(d.ms[2], d.ss[2]);
    k.Du1 = disp_interval(d.ms[6], d.ss[6]); k.Du2 = disp_interval(d.ms[7], d.ss[7]);
    k.rx = {0.0, 0.0}; k.rz = {0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 5; ++q) k.R[q] = iv(0.0f, 0.0f);
    k.unb = 0;
    if (!springs) return;
    SpringSetup st;
    spring_setup_v(d.zs[0], d.zs[1], d.zj[0], d.zj[1], k.Dx, k.Dz, disp_interval(d.mj[0], d.sj[0]),
                   disp_interval(d.mj[1], d.sj[1]), K.L0, st);
    AccPrimal acc;
    SpringPieces pc;
    const bool ok = spring_core<false>(st.dxA, st.dxB, st.dz0, st.dz1, st.dz2, st.Dxi, st.Dzi, st.Dxj,
                                                  st.Dzj, maskv(st.Dxi), maskv(st.Dzi), maskv(st.Dxj),
                                                  maskv(st.Dzj), K.K3, K.K15, K.K1, K.K05, acc, pc);
    k.unb = right && !ok ? 1u : 0u;
    // (an unbounded spring's values are never used: its rows are infinite)
    const double rxl = acc.a[S_CX].lo + acc.a[S_BX].lo, rxh = acc.a[S_CX].hi + acc.a[S_BX].hi;
    const double rzl = acc.a[S_CZ].lo + acc.a[S_BZ].lo, rzh = acc.a[S_CZ].hi + acc.a[S_BZ].hi;
    k.rx.lo = right ? rxl : 0.0; k.rx.hi = right ? rxh : 0.0;
    k.rz.lo = right ? rzl : 0.0; k.rz.hi = right ? rzh : 0.0;
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        k.R[q].lo = right ? pc.R[q].lo : 0.0f;
        k.R[q].hi = right ? pc.R[q].hi : 0.0f;
    }
    if (right) {
        // row i+1 receives -(cross + node i's own pairs)
        out->xlo = -(acc.a[S_CX].hi + acc.a[S_AX].hi); out->xhi = -(acc.a[S_CX].lo + acc.a[S_AX].lo);
        out->zlo = -(acc.a[S_CZ].hi + acc.a[S_AZ].hi); out->zhi = -(acc.a[S_CZ].lo + acc.a[S_AZ].lo);
#pragma unroll
        for (int q = 0; q < 5; ++q) out->L[q] = pc.L[q];
        out->unbounded = k.unb;
    }
}

// Node i: attitude block, the left spring's terms (left == NULL for node 0),
// shared position pairs.  ft: the timestep's flags.  Rows 3 and 4 of the
// node as [lo3, hi3], [lo4, hi4]; a bad input makes every row of the node
// (-inf, inf) (*all_inf = true), an unbounded spring rows 3 and 4.
__device__ __forceinline__ void node_step(const NodeConsts& K, int U, const NodeIn& d, const SpringKeep& k,
                                          const SpringOut* left, uint32_t ft, double* lo34, double* hi34,
                                          bool* all_inf) {
    IV<float> L[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) L[q] = iv(0.0f, 0.0f);
    div_ ox = k.rx, oz = k.rz;
    uint32_t row_unb = k.unb;
    if (left) {
        row_unb |= left->unbounded;
        ox.lo += left->xlo; ox.hi += left->xhi; oz.lo += left->zlo; oz.hi += left->zhi;
#pragma unroll
        for (int q = 0; q < 5; ++q) L[q] = left->L[q];
    }
    NodeTerms nt;
    node_terms(d.zs[2], d.vs[0] + d.vs[1], k.Dth, k.Du1, k.Du2, k.Dx, k.Dz, k.R, L, U > 1 && !row_unb, K.c, K.K15,
               K.K1, K.K05, maskv(k.Dth), maskv(k.Du1), maskv(k.Du2), maskv(k.Dx), maskv(k.Dz), nt);
#pragma unroll
    for (int q = 0; q < 12; ++q) {
        div_& acc = node_term_row(q) == 0 ? ox : oz;
        const float a = nt.neg[q] ? nt.T[q].hi : nt.T[q].lo;
        const float b = nt.neg[q] ? nt.T[q].lo : nt.T[q].hi;
        acc.lo = __builtin_fma(nt.k[q], (double)a, acc.lo);
        acc.hi = __builtin_fma(nt.k[q], (double)b, acc.hi);
    }
    *all_inf = (ft & LEB_FLAG_BAD_INPUT) != 0u;
    if (*all_inf || row_unb) {
        lo34[0] = lo34[1] = -INFINITY; hi34[0] = hi34[1] = INFINITY;
    } else {
        // all lower-end summands are <= 0 and all upper-end summands >= 0,
        // so 2^-45 relative covers every FP64 rounding in the sums
        lo34[0] = wlo64(ox.lo); hi34[0] = whi64(ox.hi); lo34[1] = wlo64(oz.lo); hi34[1] = whi64(oz.hi);
    }
}

// zonotope packaging of a row [lo, hi] (eq. zono_map): centre, radius + pad
__device__ __forceinline__ void row_zono(double lo, double hi, double pad, double* cb, double* rb) {
    if (isfinite(lo) && isfinite(hi)) {
        *cb = 0.5 * (lo + hi);
        double r = fmax(hi - *cb, *cb - lo);
        *rb = r + fabs(r) * 0x1p-50 + pad;
    } else {
        *cb = 0.0;
        *rb = INFINITY;
    }
}

// Orders one wave's own LDS accesses (its lanes exchange values without the
// other waves of the workgroup).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Spring i and node i of timestep lt; s_sp [T][U], s_flag [T] (cleared).
// Contains one workgroup barrier (ONE_WAVE: none, the timestep's nodes are lanes
// of the one calling wave).  Args supplies U, c (dt/m), kL, L0, pad and
// compact (1: c_bar, rho_bar hold rows 3 and 4 of each node only).
template <bool ONE_WAVE = false, class Args>
__device__ __forceinline__ void node_pass(const Args& A, const TileRef& t, const NodeIn& d, int lt, int i,
                                          SpringOut* s_sp, uint32_t* s_flag) {
    const int U = A.U, nx = 6 * U;
    const bool active = lt < t.nloc;
    const bool right = active && i < U - 1;      // spring i exists
    if (active) {
        const uint32_t f = node_flags(d);
        if (f) atomicOr(&s_flag[lt], f);
    }
    const NodeConsts K = node_consts(A.c, A.kL, A.L0);
    SpringKeep k;
    spring_step(K, d, U > 1, right, k, &s_sp[lt * U + i]);
    if (k.unb) atomicOr(&s_flag[lt], LEB_FLAG_UNBOUNDED);
    if (ONE_WAVE) wave_lds_fence();
    else __syncthreads();      // spring terms and flags complete
    if (!active) return;
    const uint32_t ft = s_flag[lt];
    double lo34[2], hi34[2];
    bool all_inf;
    node_step(K, U, d, k, i > 0 ? &s_sp[lt * U + i - 1] : nullptr, ft, lo34, hi34, &all_inf);
    double lo[6], hi[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        lo[c] = all_inf ? -INFINITY : 0.0;
        hi[c] = all_inf ? INFINITY : 0.0;
    }
    lo[3] = lo34[0]; hi[3] = hi34[0]; lo[4] = lo34[1]; hi[4] = hi34[1];
    const int64_t o = (int64_t)lt * nx + 6 * i;
    auto put = [](double* p, double x, double y) { *reinterpret_cast<node_d2*>(p) = node_d2{x, y}; };
    if (t.RLO) {
#pragma unroll
        for (int c = 0; c < 6; c += 2) { put(t.RLO + o + c, lo[c], lo[c + 1]); put(t.RHI + o + c, hi[c], hi[c + 1]); }
    }
    if (t.CB) {
        double cb[6], rb[6];
        // compact: the four affine rows are exactly (0, pad) unless the unit is bad, and
        // then rows 3 and 4 are not finite either
        if (A.compact) {
            const int64_t o2 = 2 * ((int64_t)lt * U + i);
            row_zono(lo[3], hi[3], A.pad, &cb[3], &rb[3]);
            row_zono(lo[4], hi[4], A.pad, &cb[4], &rb[4]);
            put(t.CB + o2, cb[3], cb[4]);
            put(t.RB + o2, rb[3], rb[4]);
        } else {
#pragma unroll
            for (int c = 0; c < 6; ++c) row_zono(lo[c], hi[c], A.pad, &cb[c], &rb[c]);
#pragma unroll
            for (int c = 0; c < 6; c += 2) { put(t.CB + o + c, cb[c], cb[c + 1]); put(t.RB + o + c, rb[c], rb[c + 1]); }
        }
    }
    if (t.FL && i == 0) t.FL[lt] = (ft & LEB_FLAG_BAD_INPUT) ? (ft & ~LEB_FLAG_UNBOUNDED) : ft;
}

}  // namespace leb
