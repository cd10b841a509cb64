// smalldyn.hip -- interval-Hessian bounds of small analytic systems: the
// closed-form test dynamics (LINEAR, QUADRATIC,
// SINCOS), the satellite and the 3-D quadrotor of the dynamics appendix,
// each in the three forms the paper compares (section IV.A):
//   PATH     Theorem 1: sum_{j<k} [H_kj](X^(j)) (Delta_j Delta_k)
//                       + 1/2 sum_k [H_kk](X^(k)) Delta_k^2, prefix boxes X^(p)
//   EXPAND   eq. expanded_interval_hessian: the same sum, every entry over X
//   CLASSIC  eq. interval_quadratic_form: 1/2 Delta^T ([H](X) Delta)
// and the random-sampling under-approximation of the remainder (the
// comparison of the tightness study): min and max of r(a; a~) over
// caller-given points of the box.
//
// Arithmetic as in the chain kernel: the displacement intervals and the
// Hessian entries in outward-rounded FP32, every entry times an FP64 point
// factor (dt, a quadratic coefficient), the terms summed in FP64.  Every
// term contains 0 (each has a displacement factor that does), so the FP64
// sums do not cancel and one relative widening covers their rounding.  A
// term whose displacement factor is exactly [0, 0] contributes exactly 0.
#include <hip/hip_runtime.h>
#include <float.h>
#include <math.h>
#include <stdint.h>

#include "leb.h"
#include "leb_internal.hpp"
#include "pbh_common.hpp"
#include "pbh_node.hpp"

namespace leb {

constexpr int SD_MAX_N = 64;     // QUADRATIC: nx + nu
constexpr int SD_MAX_CAND = 9;   // structural entries of one row (3-D quadrotor: velocity rows)

struct SmallArgs {
    const double *z, *v, *mu, *sigma, *Q;
    double *r_lo, *r_hi, *c_bar, *rho_bar;
    uint32_t* flags;
    double pad;
    int64_t units;
    int nx, nu, kind;
    double dt, m, J[3];
};

__device__ __forceinline__ double sd_nom(const SmallArgs& A, int64_t u, int i) {
    return i < A.nx ? A.z[u * A.nx + i] : A.v[u * A.nu + (i - A.nx)];
}
__device__ __forceinline__ fiv sd_disp(const SmallArgs& A, int64_t u, int i) {
    const int n = A.nx + A.nu;
    const IV<float> d = disp_interval(A.mu ? A.mu[u * n + i] : 0.0, A.sigma[u * n + i]);
    return mk(d.lo, d.hi);
}
__device__ __forceinline__ bool sd_zero(fiv d) { return d.lo == 0.0f && d.hi == 0.0f; }

// Coordinate i of the prefix box X^(p) (coordinates 0..p free, the rest at
// the nominal), FP64 endpoints rounded outward.
__device__ __forceinline__ void sd_coord(const SmallArgs& A, int64_t u, int i, int p, double* lo, double* hi) {
    const double a = sd_nom(A, u, i);
    if (i > p) { *lo = a; *hi = a; return; }
    const fiv d = sd_disp(A, u, i);
    const double l = a + (double)d.lo, h = a + (double)d.hi;
    *lo = l - fabs(l) * 0x1p-52;
    *hi = h + fabs(h) * 0x1p-52;
}
__device__ __forceinline__ fiv sd_coord32(const SmallArgs& A, int64_t u, int i, int p) {
    double lo, hi;
    sd_coord(A, u, i, p, &lo, &hi);
    return mk(rd32(lo), ru32(hi));
}
__device__ __forceinline__ SinCos sd_trig(const SmallArgs& A, int64_t u, int i, int p) {
    double lo, hi;
    sd_coord(A, u, i, p, &lo, &hi);
    SinCos r;
    isincos(lo, hi, &r);
    return r;
}

// --------------------------------------------------------------- entries
//
// An entry is kappa * H: kappa an FP64 point, H an FP32 interval (unit when
// `unit` is set, so that a point coefficient is applied once, in FP64).
struct Entry {
    fiv H;
    double kappa;
    bool unit;
};

// Satellite: qdot_r = sum over (w_b, q_c) of +-1/2 w_b q_c (zeta carries the
// 1/2); wdot_1 = ... - (I3 - I2)/I1 w2 w3 and cyclically.  a = (q0..q3, w1..w3, v1..v3).
constexpr signed char kSatQ[4][3][3] = {
    {{1, 1, -1}, {2, 2, -1}, {3, 3, -1}},
    {{1, 0, 1}, {3, 2, 1}, {2, 3, -1}},
    {{2, 0, 1}, {3, 1, -1}, {1, 3, 1}},
    {{3, 0, 1}, {2, 1, 1}, {1, 2, -1}}};

__device__ __forceinline__ double sat_euler(const SmallArgs& A, int r) {    // -(I_b - I_c)/I_a dt, a = r
    const int b = r == 0 ? 2 : (r == 1 ? 0 : 1), c = r == 0 ? 1 : (r == 1 ? 2 : 0);
    return -A.dt * (A.J[b] - A.J[c]) / A.J[r];
}

// 3-D quadrotor: a = (px, py, pz, phi, theta, psi, vx, vy, vz, p, q, r, T, tau x3)
enum { QD_PHI = 3, QD_TH = 4, QD_PSI = 5, QD_P = 9, QD_Q = 10, QD_R = 11, QD_T = 12 };

// The structurally non-zero entries (k, j), k >= j, of each row (-1: none left).
__constant__ signed char kQuad3dEntries[12][SD_MAX_CAND][2] = {
    {{-1, -1}}, {{-1, -1}}, {{-1, -1}},
    {{3, 3}, {10, 3}, {11, 3}, {4, 3}, {4, 4}, {10, 4}, {11, 4}, {-1, -1}, {-1, -1}},
    {{3, 3}, {10, 3}, {11, 3}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}},
    {{3, 3}, {10, 3}, {11, 3}, {4, 3}, {4, 4}, {10, 4}, {11, 4}, {-1, -1}, {-1, -1}},
    {{3, 3}, {4, 3}, {4, 4}, {12, 3}, {12, 4}, {5, 3}, {5, 4}, {5, 5}, {12, 5}},
    {{3, 3}, {4, 3}, {4, 4}, {12, 3}, {12, 4}, {5, 3}, {5, 4}, {5, 5}, {12, 5}},
    {{3, 3}, {4, 3}, {4, 4}, {12, 3}, {12, 4}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}},
    {{11, 10}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}},
    {{11, 9}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}},
    {{10, 9}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}}};

// entry c of row l; false past the row's last one
__device__ __forceinline__ bool sd_candidate(const SmallArgs& A, int l, int c, int* k, int* j) {
    *k = *j = 0;
    if (A.kind == LEB_DYN_SINCOS) {
        if (c >= (A.nx == 2 ? 3 : 1)) return false;
        *k = c > 0;
        *j = c > 1;
        return true;
    }
    if (A.kind == LEB_DYN_SATELLITE) {
        if (c >= (l < 4 ? 3 : 1)) return false;
        if (l < 4) { *k = 3 + kSatQ[l][c][0]; *j = kSatQ[l][c][1]; }
        else { *k = l == 6 ? 5 : 6; *j = l == 4 ? 5 : 4; }
        return true;
    }
    if (l < 3 || c >= SD_MAX_CAND || kQuad3dEntries[l][c][0] < 0) return false;
    *k = kQuad3dEntries[l][c][0];
    *j = kQuad3dEntries[l][c][1];
    return true;
}

// The 3-D quadrotor's entries see phi over its interval (every entry's prefix
// includes phi), theta, psi, q, r, T either at the nominal ([0]) or over their
// intervals ([1]).
struct SinCosIv { fiv s, c; };
struct Q3Cache {
    SinCosIv phi, th[2], psi[2];
    fiv q[2], r[2], T[2];
};

// The unit's cache, one element a lane (c = 0 .. 15), written to LDS.
__device__ __forceinline__ void q3_cache(const SmallArgs& A, int64_t u, int c, Q3Cache& C) {
    const int full = A.nx + A.nu - 1;
    if (c < 5) {
        const int i = c == 0 ? QD_PHI : (c < 3 ? QD_TH : QD_PSI);
        const SinCos t = sd_trig(A, u, i, (c == 1 || c == 3) ? i - 1 : full);
        (&C.phi)[c] = SinCosIv{t.s, t.c};
    } else if (c < 11) {
        const int q = c - 5, i = q < 2 ? QD_Q : (q < 4 ? QD_R : QD_T);
        C.q[q] = sd_coord32(A, u, i, (q & 1) ? full : 0);
    }
}

// Entry (k, j) of row l over the prefix box X^(p): 1 (written to e), -1 unbounded.
__device__ int sd_entry(const SmallArgs& A, int64_t u, int l, int k, int j, int p, const Q3Cache& C, Entry& e) {
    e.unit = false;
    e.kappa = 1.0;
    if (A.kind == LEB_DYN_SINCOS) {
        // f = sin a1 (1-D); f1 = sin a1 cos a2, f2 = cos a1 sin a2 (2-D)
        const SinCos t0 = sd_trig(A, u, 0, p);
        if (A.nx == 1) { e.H = neg(t0.s); return 1; }
        const SinCos t1 = sd_trig(A, u, 1, p);
        const bool diag = k == j;
        if (l == 0) e.H = neg(diag ? mul(t0.s, t1.c) : mul(t0.c, t1.s));
        else e.H = neg(diag ? mul(t0.c, t1.s) : mul(t0.s, t1.c));
        return 1;
    }
    if (A.kind == LEB_DYN_SATELLITE) {
        e.unit = true;
        e.H = mk(1.0f, 1.0f);
        if (l < 4) {
            for (int t = 0; t < 3; ++t)
                if (k == 3 + kSatQ[l][t][0] && j == kSatQ[l][t][1]) e.kappa = 0.5 * kSatQ[l][t][2] * A.dt;
        } else {
            e.kappa = sat_euler(A, l - 4);
        }
        return 1;
    }
    // LEB_DYN_QUAD3D
    e.kappa = A.dt;
    if (l >= 9) {
        const int i = l - 9;
        const int na = i == 0 ? 1 : (i == 1 ? 2 : 0), nb = i == 0 ? 2 : (i == 1 ? 0 : 1);
        e.unit = true;
        e.H = mk(1.0f, 1.0f);
        e.kappa = A.dt * (A.J[na] - A.J[nb]) / A.J[i];
        return 1;
    }
    const fiv sf = C.phi.s, cf = C.phi.c;
    if (l <= 5) {
        const fiv q = C.q[p >= QD_Q], r = C.r[p >= QD_R];
        const fiv Aa = add(mul(q, sf), mul(r, cf));          // A = q sin(phi) + r cos(phi)
        const fiv Bb = sub(mul(q, cf), mul(r, sf));          // B = q cos(phi) - r sin(phi)
        if (l == 4) {
            e.H = k == QD_PHI ? neg(Bb) : (k == QD_Q ? neg(sf) : neg(cf));
            return 1;
        }
        const SinCosIv& tt = C.th[p >= QD_TH];
        if (!(tt.c.lo > 0.0f)) return -1;                    // sec, tan unbounded
        const fiv sec = rcp_pos(tt.c);
        const fiv tn = mul(tt.s, sec);
        const fiv sec2 = mul_nn(sec, sec);
        if (l == 3) {
            if (j == QD_PHI) {
                if (k == QD_PHI) e.H = neg(mul(Aa, tn));
                else if (k == QD_TH) e.H = mul(Bb, sec2);
                else if (k == QD_Q) e.H = mul(cf, tn);
                else e.H = neg(mul(sf, tn));
            } else {
                if (k == QD_TH) e.H = mul(mk(2.0f * Aa.lo, 2.0f * Aa.hi), mul(sec2, tn));
                else if (k == QD_Q) e.H = mul(sf, sec2);
                else e.H = mul(cf, sec2);
            }
        } else {
            const fiv st = mul(sec, tn);
            if (j == QD_PHI) {
                if (k == QD_PHI) e.H = neg(mul(Aa, sec));
                else if (k == QD_TH) e.H = mul(Bb, st);
                else if (k == QD_Q) e.H = mul(cf, sec);
                else e.H = neg(mul(sf, sec));
            } else {
                if (k == QD_TH) e.H = mul(Aa, mul(sec, add(sq(tn), sec2)));
                else if (k == QD_Q) e.H = mul(sf, st);
                else e.H = mul(cf, st);
            }
        }
        return 1;
    }
    // velocity rows: (T/m) R with R = Rx, Ry, Rz
    const SinCosIv& tt = C.th[p >= QD_TH];
    const SinCosIv& tp = C.psi[p >= QD_PSI];
    const fiv st = tt.s, ct = tt.c, sp = tp.s, cp = tp.c;
    const int r = l - 6;
    fiv D;
    if (k == QD_T) {                 // (T, b): (1/m) dR/db
        if (r == 0) {
            if (j == QD_PHI) D = sub(mul(sp, cf), mul(mul(cp, st), sf));
            else if (j == QD_TH) D = mul(mul(cp, ct), cf);
            else D = sub(mul(cp, sf), mul(mul(sp, st), cf));
        } else if (r == 1) {
            if (j == QD_PHI) D = neg(add(mul(mul(sp, st), sf), mul(cp, cf)));
            else if (j == QD_TH) D = mul(mul(sp, ct), cf);
            else D = add(mul(mul(cp, st), cf), mul(sp, sf));
        } else {
            D = j == QD_PHI ? neg(mul(ct, sf)) : neg(mul(st, cf));
        }
        e.H = D;
        e.kappa = A.dt / A.m;
        return 1;
    }
    if (r == 0) {
        if (k == QD_PHI) D = neg(add(mul(mul(cp, st), cf), mul(sp, sf)));
        else if (k == QD_TH && j == QD_PHI) D = neg(mul(mul(cp, ct), sf));
        else if (k == QD_TH) D = neg(mul(mul(cp, st), cf));
        else if (j == QD_PHI) D = add(mul(mul(sp, st), sf), mul(cp, cf));
        else if (j == QD_TH) D = neg(mul(mul(sp, ct), cf));
        else D = neg(add(mul(mul(cp, st), cf), mul(sp, sf)));
    } else if (r == 1) {
        if (k == QD_PHI) D = sub(mul(cp, sf), mul(mul(sp, st), cf));
        else if (k == QD_TH && j == QD_PHI) D = neg(mul(mul(sp, ct), sf));
        else if (k == QD_TH) D = neg(mul(mul(sp, st), cf));
        else if (j == QD_PHI) D = sub(mul(sp, cf), mul(mul(cp, st), sf));
        else if (j == QD_TH) D = mul(mul(cp, ct), cf);
        else D = sub(mul(cp, sf), mul(mul(sp, st), cf));
    } else {
        if (k == QD_PHI) D = neg(mul(ct, cf));
        else if (j == QD_PHI) D = mul(st, sf);
        else D = neg(mul(ct, cf));
    }
    e.H = mul(C.T[p >= QD_T], D);
    e.kappa = A.dt / A.m;
    return 1;
}

// kappa * H * P into acc (P contains 0)
__device__ __forceinline__ void sd_acc(div_& acc, const Entry& e, double scale, fiv P) {
    acc_any(acc, scale * e.kappa, e.unit ? P : mul_z(e.H, P));
}

// CLASSIC: coordinate i's share 1/2 Delta_i v_i (both factors contain 0, so the product does too)
__device__ __forceinline__ void sd_classic(fiv d, div_ v, div_& acc) {
    if (sd_zero(d)) return;
    acc.lo += 0.5 * fmin((double)d.lo * v.hi, (double)d.hi * v.lo);
    acc.hi += 0.5 * fmax((double)d.lo * v.lo, (double)d.hi * v.hi);
}

// a row's accumulated ends, widened, or the enclosure of an invalid or unbounded row
__device__ __forceinline__ void sd_row_out(const SmallArgs& A, int64_t u, int l, div_ acc, bool any, bool bad,
                                           bool unbounded) {
    double lo, hi;
    if (bad || unbounded) {
        lo = -INFINITY; hi = INFINITY;
    } else {
        // at most a few thousand same-sign FP64 roundings of 2^-53 each, relative to the sum
        lo = acc.lo - fabs(acc.lo) * 0x1p-40;
        hi = acc.hi + fabs(acc.hi) * 0x1p-40;
        if (!any) { lo = 0.0; hi = 0.0; }
    }
    const int64_t o = u * A.nx + l;
    if (A.r_lo) { A.r_lo[o] = lo; A.r_hi[o] = hi; }
    if (A.c_bar) row_zono(lo, hi, A.pad, &A.c_bar[o], &A.rho_bar[o]);
}

__device__ __forceinline__ uint32_t sd_input_flags(const SmallArgs& A, int64_t u, int i) {
    const int n = A.nx + A.nu;
    const double a = sd_nom(A, u, i), m = A.mu ? A.mu[u * n + i] : 0.0, s = A.sigma[u * n + i];
    uint32_t fl = 0;
    if (!isfinite(a) || !isfinite(m) || !isfinite(s) || !(s >= 0.0)) fl |= LEB_FLAG_BAD_INPUT;
    if (fabs(m) > s) fl |= LEB_FLAG_HULL_EXTENDED;
    return fl;
}

// LINEAR (G = 1, one thread writes every row of its unit) and QUADRATIC: one thread
// per (unit, row), the rows of a unit G consecutive lanes (G a power of two >= nx,
// so a group never straddles a wave); the unit's flags are OR-ed over its group.
template <int MODE>
__global__ void __launch_bounds__(256) small_poly_kernel(SmallArgs A, int G) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t u = q / G;
    const int lane_row = (int)(q - u * G);
    const bool active = u < A.units && lane_row < A.nx;
    const int n = A.nx + A.nu;
    uint32_t fl = 0, fl_row = 0;
    if (active)
        for (int i = 0; i < n; ++i) fl |= sd_input_flags(A, u, i);
    const bool bad = (fl & LEB_FLAG_BAD_INPUT) != 0;
    const int l_end = A.kind == LEB_DYN_LINEAR ? A.nx : lane_row + 1;
    for (int l = lane_row; active && l < l_end; ++l) {
        div_ vk[MODE == LEB_IH_CLASSIC ? SD_MAX_N : 1];
        div_ acc{0.0, 0.0};
        int terms = 0;
        bool unbounded = false;
        if (!bad && A.kind != LEB_DYN_LINEAR) {
            if (MODE == LEB_IH_CLASSIC)
                for (int i = 0; i < n; ++i) vk[i] = div_{0.0, 0.0};
            const double* Ql = A.Q + (size_t)l * n * n;
            for (int k = 0; k < n && !unbounded; ++k)
                for (int j = 0; j <= k; ++j) {
                    const double qv = Ql[k * n + j];
                    if (!isfinite(qv)) { unbounded = true; break; }
                    if (qv == 0.0) continue;
                    Entry e;
                    e.unit = true; e.H = mk(1.0f, 1.0f); e.kappa = qv;
                    const fiv dk = sd_disp(A, u, k), dj = sd_disp(A, u, j);
                    if (MODE == LEB_IH_CLASSIC) {
                        // v = [H] Delta over the symmetric matrix: row k gets H Delta_j, row j gets H Delta_k
                        if (!sd_zero(dj)) { sd_acc(vk[k], e, 1.0, dj); ++terms; }
                        if (k != j && !sd_zero(dk)) { sd_acc(vk[j], e, 1.0, dk); ++terms; }
                    } else if (!sd_zero(dk) && !sd_zero(dj)) {
                        if (j < k) sd_acc(acc, e, 1.0, mul_zz(dj, dk));
                        else sd_acc(acc, e, 0.5, sq_z(dk));
                        ++terms;
                    }
                }
            if (MODE == LEB_IH_CLASSIC && !unbounded)
                for (int i = 0; i < n; ++i) sd_classic(sd_disp(A, u, i), vk[i], acc);
        }
        if (unbounded) fl_row = LEB_FLAG_UNBOUNDED;
        sd_row_out(A, u, l, acc, terms != 0, bad, unbounded);
    }
    // every lane takes part in the exchange; inactive lanes contribute 0
    uint32_t f = fl | fl_row;
    for (int off = 1; off < G; off <<= 1) f |= (uint32_t)__shfl_xor((int)f, off);
    if (active && lane_row == 0 && A.flags) A.flags[u] = f;
}

// SINCOS, SATELLITE and QUAD3D: a wave bounds one row of 64 / G units, lane (unit, c)
// one Hessian entry of the row, so the row's entries run side by side and the rows of a
// unit on different waves; the 3-D quadrotor's trigonometric enclosures are computed one a
// lane and shared through LDS.  CLASSIC sums v = [H] Delta per coordinate: lane c of the
// unit's G collects the entries that touch coordinates c, c + G, ...
//
// G is the most entries that a row of the system has, up to a power of two: 16 for the 3-D
// quadrotor (9), 4 for the satellite and SINCOS in two dimensions (3), 1 for SINCOS in
// one.  What bounds it is latency up to some thousand units (a serial chain of interval
// operations, one wave a row: PATH, EXPAND, CLASSIC of one local set of the 3-D quadrotor
// 9.3, 9.7 and 11 us, one thread per row and its entries one after the other 24, 22 and
// 30 us), then the instructions issued, of which lanes without an entry take their share.
// Many units, PATH, whole call: satellite x 400,000 107 us (one thread per row 190, 16 lanes
// a row 354), SINCOS x 1,000,000 in two dimensions 189 us (277, 725), in one 21 us (47, 224),
// 3-D quadrotor x 400,000 1,080 us (1,190 and the same 1,080).
template <int MODE, int KIND, int G>
__global__ void __launch_bounds__(256) small_entry_kernel(SmallArgs A) {
    constexpr bool Q3 = KIND == LEB_DYN_QUAD3D;
    // (not a changed copy of A: J is indexed, and a copy would lie in scratch)
    __builtin_assume(A.kind == KIND);
    __shared__ div_ s_v[4][64][2];           // CLASSIC: entry c's contributions to v_k and v_j
    __shared__ signed char s_kj[4][64][2];
    __shared__ Q3Cache s_q3[4][Q3 ? 64 / G : 1];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t wid = (int64_t)blockIdx.x * 4 + wave;
    const int64_t ug = wid / A.nx;
    const int l = (int)(wid - ug * A.nx), c = lane & (G - 1), first = lane & ~(G - 1);
    const int64_t u = (64 / G) * ug + lane / G;
    const bool active = u < A.units;
    const int n = A.nx + A.nu, full = n - 1;          // X^(n-1) = X
    Q3Cache& C = s_q3[wave][Q3 ? lane / G : 0];
    const uint64_t group = ((1ull << G) - 1ull) << first;
    // the unit's flags, the coordinates shared out over its lanes
    uint32_t mine = 0u;
    if (active)
        for (int i = c; i < n; i += G) mine |= sd_input_flags(A, u, i);
    const bool bad = (__ballot(mine & LEB_FLAG_BAD_INPUT) & group) != 0;
    const bool hull = (__ballot(mine & LEB_FLAG_HULL_EXTENDED) & group) != 0;
    div_ acc{0.0, 0.0};
    bool unb = false, any = false;
    int k = 0, j = 0;
    const bool entry = active && !bad && sd_candidate(A, l, c, &k, &j);
    if (Q3) {
        if (active && !bad && (l == 0 || (l >= 3 && l <= 8))) q3_cache(A, u, c, C);
        wave_lds_fence();
    }
    if (entry) {
        Entry e;
        unb = sd_entry(A, u, l, k, j, MODE == LEB_IH_PATH ? j : full, C, e) < 0;     // prefix of the smaller index
        const fiv dk = sd_disp(A, u, k), dj = sd_disp(A, u, j);
        if (MODE == LEB_IH_CLASSIC) {
            // v = [H] Delta over the symmetric matrix: row k gets H Delta_j, row j gets H Delta_k
            div_ vk{0.0, 0.0}, vj{0.0, 0.0};
            if (!unb && !sd_zero(dj)) { sd_acc(vk, e, 1.0, dj); any = true; }
            if (!unb && k != j && !sd_zero(dk)) { sd_acc(vj, e, 1.0, dk); any = true; }
            s_v[wave][lane][0] = vk;
            s_v[wave][lane][1] = vj;
        } else if (!unb && !sd_zero(dk) && !sd_zero(dj)) {
            if (j < k) sd_acc(acc, e, 1.0, mul_zz(dj, dk));
            else sd_acc(acc, e, 0.5, sq_z(dk));
            any = true;
        }
    }
    if (MODE == LEB_IH_CLASSIC) {
        s_kj[wave][lane][0] = entry ? (signed char)k : (signed char)-1;
        s_kj[wave][lane][1] = entry && k != j ? (signed char)j : (signed char)-1;
        wave_lds_fence();
        if (active && !bad)
            for (int i = c; i < n; i += G) {
                div_ v{0.0, 0.0};
                for (int q = 0; q < (G < SD_MAX_CAND ? G : SD_MAX_CAND); ++q) {
                    const int o = first + q;
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        if (s_kj[wave][o][h] == i) { v.lo += s_v[wave][o][h].lo; v.hi += s_v[wave][o][h].hi; }
                }
                sd_classic(sd_disp(A, u, i), v, acc);
            }
    }
    // sums over the lanes of the unit (every lane takes part)
#pragma unroll
    for (int off = 1; off < G; off <<= 1) {
        acc.lo += __shfl_xor(acc.lo, off);
        acc.hi += __shfl_xor(acc.hi, off);
    }
    const bool row_any = (__ballot(any) & group) != 0, row_unb = (__ballot(unb) & group) != 0;
    if (active && c == 0) sd_row_out(A, u, l, acc, row_any, bad, row_unb);
    if (A.flags && l == 0 && active && c == 0) {
        // row 0's wave reports the unit: only the 3-D quadrotor's attitude rows can be
        // unbounded, where cos(theta) over the widest theta they see is not positive
        uint32_t f = (bad ? LEB_FLAG_BAD_INPUT : 0u) | (hull ? LEB_FLAG_HULL_EXTENDED : 0u);
        if (Q3 && !bad && (!(C.th[1].c.lo > 0.0f) || (MODE == LEB_IH_PATH && !(C.th[0].c.lo > 0.0f))))
            f |= LEB_FLAG_UNBOUNDED;
        A.flags[u] = f;
    }
}

template <int KIND, int G>
static int launch_small_entry(int mode, const SmallArgs& A, hipStream_t s) {
    const int64_t blocks = ((A.units + 64 / G - 1) / (64 / G) * A.nx + 3) / 4;      // a wave per row of 64 / G units
    if (blocks > 0x7fffffff) return LEB_EINVAL;
    const dim3 g((unsigned)blocks), b(256);
    if (mode == LEB_IH_PATH) hipLaunchKernelGGL((small_entry_kernel<LEB_IH_PATH, KIND, G>), g, b, 0, s, A);
    else if (mode == LEB_IH_EXPAND) hipLaunchKernelGGL((small_entry_kernel<LEB_IH_EXPAND, KIND, G>), g, b, 0, s, A);
    else hipLaunchKernelGGL((small_entry_kernel<LEB_IH_CLASSIC, KIND, G>), g, b, 0, s, A);
    return LEB_OK;
}

// --------------------------------------------------- sampled remainder
//
// r_l(a; a~) = N_l(a) - N_l(a~) - grad N_l(a~) . (a - a~), N the non-affine
// part of the dynamics, in FP64; QUADRATIC uses its exact form 1/2 d^T Q_l d.

constexpr int SD_SAMPLE_N = 16;      // nx + nu of the sampled kinds

// N_l(a) for every row l < nx at once (each trigonometric value computed once)
__device__ __forceinline__ void sd_nonlin_all(const SmallArgs& A, const double (&a)[SD_SAMPLE_N],
                                              double (&N)[SD_SAMPLE_N]) {
#pragma unroll
    for (int l = 0; l < SD_SAMPLE_N; ++l) N[l] = 0.0;
    if (A.kind == LEB_DYN_SINCOS) {
        if (A.nx == 1) { N[0] = sin(a[0]); return; }
        const double s0 = sin(a[0]), c0 = cos(a[0]), s1 = sin(a[1]), c1 = cos(a[1]);
        N[0] = s0 * c1;
        N[1] = c0 * s1;
        return;
    }
    if (A.kind == LEB_DYN_SATELLITE) {
#pragma unroll
        for (int l = 0; l < 4; ++l)
#pragma unroll
            for (int t = 0; t < 3; ++t)
                N[l] += 0.5 * kSatQ[l][t][2] * A.dt * a[3 + kSatQ[l][t][0]] * a[kSatQ[l][t][1]];
        N[4] = sat_euler(A, 0) * a[6] * a[5];
        N[5] = sat_euler(A, 1) * a[6] * a[4];
        N[6] = sat_euler(A, 2) * a[5] * a[4];
        return;
    }
    // LEB_DYN_QUAD3D
    const double dt = A.dt;
    double sf, cf, st, ct, sp, cp;
    sincos(a[QD_PHI], &sf, &cf);
    sincos(a[QD_TH], &st, &ct);
    sincos(a[QD_PSI], &sp, &cp);
    const double q = a[QD_Q], r = a[QD_R];
    const double Aa = q * sf + r * cf, Bb = q * cf - r * sf;
    N[3] = dt * Aa * (st / ct);
    N[4] = dt * Bb;
    N[5] = dt * Aa / ct;
    const double c = dt * a[QD_T] / A.m;
    N[6] = c * (cp * st * cf + sp * sf);
    N[7] = c * (sp * st * cf - cp * sf);
    N[8] = c * (ct * cf);
    N[9] = dt * (A.J[1] - A.J[2]) / A.J[0] * a[QD_R] * a[QD_Q];
    N[10] = dt * (A.J[2] - A.J[0]) / A.J[1] * a[QD_R] * a[QD_P];
    N[11] = dt * (A.J[0] - A.J[1]) / A.J[2] * a[QD_Q] * a[QD_P];
}

struct SampleArgs {
    SmallArgs S;
    const double* t;      // [K][n] in [-1, 1]
    int K;
    double *s_lo, *s_hi;  // [units][nx]
};

// The coordinates that row l of N depends on, ascending (-1: none left): the others'
// derivatives are exactly 0.
template <int KIND> struct SampleRows;
template <> struct SampleRows<LEB_DYN_SINCOS> {
    static constexpr int NX = 2, N = 2;
    static constexpr signed char at[2][6] = {{0, 1, -1, -1, -1, -1}, {0, 1, -1, -1, -1, -1}};
};
template <> struct SampleRows<LEB_DYN_SATELLITE> {
    static constexpr int NX = 7, N = 10;
    static constexpr signed char at[7][6] = {{1, 2, 3, 4, 5, 6},    {0, 2, 3, 4, 5, 6},     {0, 1, 3, 4, 5, 6},
                                             {0, 1, 2, 4, 5, 6},    {5, 6, -1, -1, -1, -1}, {4, 6, -1, -1, -1, -1},
                                             {4, 5, -1, -1, -1, -1}};
};
template <> struct SampleRows<LEB_DYN_QUAD3D> {
    static constexpr int NX = 12, N = 16;
    static constexpr signed char at[12][6] = {{-1, -1, -1, -1, -1, -1}, {-1, -1, -1, -1, -1, -1}, {-1, -1, -1, -1, -1, -1},
                                              {3, 4, 10, 11, -1, -1},   {3, 10, 11, -1, -1, -1},  {3, 4, 10, 11, -1, -1},
                                              {3, 4, 5, 12, -1, -1},    {3, 4, 5, 12, -1, -1},    {3, 4, 5, 12, -1, -1},
                                              {10, 11, -1, -1, -1, -1}, {9, 11, -1, -1, -1, -1},  {9, 10, -1, -1, -1, -1}};
};
template <> struct SampleRows<LEB_DYN_QUADRATIC> { static constexpr int NX = SD_SAMPLE_N, N = SD_SAMPLE_N; };

// N and its non-zero derivatives (the order of SampleRows) at the nominal
template <int KIND>
__device__ __forceinline__ void sample_nominal(const SmallArgs& A, const double (&a)[SD_SAMPLE_N],
                                               double (&f)[SD_SAMPLE_N], double (&g)[SampleRows<KIND>::NX][6]) {
    sd_nonlin_all(A, a, f);
#pragma unroll
    for (int l = 0; l < SampleRows<KIND>::NX; ++l)
#pragma unroll
        for (int q = 0; q < 6; ++q) g[l][q] = 0.0;
    const double dt = A.dt;
    if constexpr (KIND == LEB_DYN_SINCOS) {
        if (A.nx == 1) { g[0][0] = cos(a[0]); return; }
        const double s0 = sin(a[0]), c0 = cos(a[0]), s1 = sin(a[1]), c1 = cos(a[1]);
        g[0][0] = c0 * c1; g[0][1] = -s0 * s1;
        g[1][0] = -s0 * s1; g[1][1] = c0 * c1;
    } else if constexpr (KIND == LEB_DYN_SATELLITE) {
#pragma unroll
        for (int l = 0; l < 4; ++l)
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const int w = 3 + kSatQ[l][t][0], q = kSatQ[l][t][1];
                const double c = 0.5 * kSatQ[l][t][2] * dt;
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    if (SampleRows<KIND>::at[l][i] == w) g[l][i] = c * a[q];
                    if (SampleRows<KIND>::at[l][i] == q) g[l][i] = c * a[w];
                }
            }
        g[4][0] = sat_euler(A, 0) * a[6]; g[4][1] = sat_euler(A, 0) * a[5];
        g[5][0] = sat_euler(A, 1) * a[6]; g[5][1] = sat_euler(A, 1) * a[4];
        g[6][0] = sat_euler(A, 2) * a[5]; g[6][1] = sat_euler(A, 2) * a[4];
    } else if constexpr (KIND == LEB_DYN_QUAD3D) {
        double sf, cf, st, ct, sp, cp;
        sincos(a[QD_PHI], &sf, &cf);
        sincos(a[QD_TH], &st, &ct);
        sincos(a[QD_PSI], &sp, &cp);
        const double q = a[QD_Q], r = a[QD_R], Aa = q * sf + r * cf, Bb = q * cf - r * sf, tn = st / ct;
        g[3][0] = dt * Bb * tn; g[3][1] = dt * Aa / (ct * ct); g[3][2] = dt * sf * tn; g[3][3] = dt * cf * tn;
        g[4][0] = -dt * Aa; g[4][1] = dt * cf; g[4][2] = -dt * sf;
        g[5][0] = dt * Bb / ct; g[5][1] = dt * Aa * st / (ct * ct); g[5][2] = dt * sf / ct; g[5][3] = dt * cf / ct;
        const double c = dt * a[QD_T] / A.m;
        g[6][0] = c * (sp * cf - cp * st * sf); g[6][1] = c * (cp * ct * cf); g[6][2] = c * (cp * sf - sp * st * cf);
        g[7][0] = c * -(sp * st * sf + cp * cf); g[7][1] = c * (sp * ct * cf); g[7][2] = c * (cp * st * cf + sp * sf);
        g[8][0] = c * (-ct * sf); g[8][1] = c * (-st * cf);
        g[6][3] = dt * (cp * st * cf + sp * sf) / A.m;
        g[7][3] = dt * (sp * st * cf - cp * sf) / A.m;
        g[8][3] = dt * (ct * cf) / A.m;
        const double c9 = dt * (A.J[1] - A.J[2]) / A.J[0], c10 = dt * (A.J[2] - A.J[0]) / A.J[1],
                     c11 = dt * (A.J[0] - A.J[1]) / A.J[2];
        g[9][0] = c9 * a[QD_R]; g[9][1] = c9 * a[QD_Q];
        g[10][0] = c10 * a[QD_R]; g[10][1] = c10 * a[QD_P];
        g[11][0] = c11 * a[QD_Q]; g[11][1] = c11 * a[QD_P];
    }
}

// bit patterns of doubles of one sign order like their magnitudes
__device__ __forceinline__ void atomic_grow(double* p, double x) {
    atomicMax(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__double_as_longlong(x));
}

__global__ void __launch_bounds__(256) sample_zero_kernel(double* lo, double* hi, int64_t cnt) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < cnt) { lo[q] = 0.0; hi[q] = 0.0; }
}

// Workgroup (unit, part): the nominal's values and gradients and every row's running
// minimum and maximum in registers, each thread a stride of the part's samples,
// combined across the wave and then the four waves.  The nominal itself
// counts as a sample (r = 0), so lo <= 0 <= hi: with several parts a unit the results
// start at 0 and the parts grow them by atomic maxima of the magnitudes, whose order
// does not matter.  The linear part sums only the coordinates that a row depends
// on (the others would add exact zeros, or NaN where their offset is not finite).
//
// What bounds it: one sample costs about 400 FP64 instructions (six sine and cosine
// values for the 3-D quadrotor), so 10,000 samples of one unit are 40 a thread in one
// workgroup, and one a thread over 40 parts.  One set of the 3-D
// quadrotor, 10,000 samples: 11 us and 1.4 us to clear (one workgroup with the kind and
// the rows chosen in the inner loops: 325 us).
template <int KIND>
__global__ void __launch_bounds__(256, 2) sample_rem_kernel(SampleArgs P, int parts) {
    using Rows = SampleRows<KIND>;
    constexpr int NX = Rows::NX, NC = Rows::N;
    const SmallArgs A = [&] { SmallArgs s = P.S; s.kind = KIND; return s; }();
    const int64_t u = blockIdx.x;
    constexpr bool FIXED = KIND == LEB_DYN_SATELLITE || KIND == LEB_DYN_QUAD3D;      // one size each
    const int n = FIXED ? NC : A.nx + A.nu, nx = FIXED ? NX : A.nx;
    __shared__ double wlo[4][SD_SAMPLE_N], whi[4][SD_SAMPLE_N];
    double a0[SD_SAMPLE_N], ctr[NC], sg[NC];
#pragma unroll
    for (int i = 0; i < SD_SAMPLE_N; ++i) a0[i] = i < n ? sd_nom(A, u, i) : 0.0;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        ctr[i] = i < n ? a0[i] + (A.mu ? A.mu[u * n + i] : 0.0) : 0.0;
        sg[i] = i < n ? A.sigma[u * n + i] : 0.0;
    }
    double f0[SD_SAMPLE_N], g0[NX][6];
    if constexpr (KIND != LEB_DYN_QUADRATIC) sample_nominal<KIND>(A, a0, f0, g0);
    double lo[NX], hi[NX];
#pragma unroll
    for (int l = 0; l < NX; ++l) { lo[l] = 0.0; hi[l] = 0.0; }
    const int64_t stride = (int64_t)parts * blockDim.x;      // (K up to 2^31 - 1: 32 bits would wrap past it)
    for (int64_t s = (int64_t)blockIdx.y * blockDim.x + threadIdx.x; s < P.K; s += stride) {
        double a[SD_SAMPLE_N], d[NC];
        uint32_t wild = 0;               // coordinates with a non-finite offset
#pragma unroll
        for (int i = 0; i < SD_SAMPLE_N; ++i) a[i] = 0.0;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            a[i] = i < n ? ctr[i] + P.t[s * n + i] * sg[i] : 0.0;
            d[i] = a[i] - a0[i];
            wild |= isfinite(d[i]) ? 0u : 1u << i;
        }
        if constexpr (KIND == LEB_DYN_QUADRATIC) {
            for (int l = 0; l < nx; ++l) {
                const double* Ql = A.Q + (size_t)l * n * n;
                double acc = 0.0;
                for (int k = 0; k < n; ++k) {
                    double row = 0.5 * Ql[k * n + k] * d[k];
                    for (int j = 0; j < k; ++j) row += Ql[k * n + j] * d[j];
                    acc += row * d[k];
                }
                lo[l] = fmin(lo[l], acc);
                hi[l] = fmax(hi[l], acc);
            }
        } else {
            double r[SD_SAMPLE_N];
            sd_nonlin_all(A, a, r);
#pragma unroll
            for (int l = 0; l < NX; ++l) {
                if (l >= nx) break;
                double lin = 0.0;
                uint32_t seen = 0;
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    const int i = Rows::at[l][q];
                    if (i >= 0) { lin += g0[l][q] * d[i]; seen |= 1u << i; }
                }
                if (wild & ~seen) lin = NAN;
                const double rv = (r[l] - f0[l]) - lin;
                lo[l] = fmin(lo[l], rv);
                hi[l] = fmax(hi[l], rv);
            }
        }
    }
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int l = 0; l < NX; ++l) {
        double x = lo[l], y = hi[l];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            x = fmin(x, __shfl_xor(x, off));
            y = fmax(y, __shfl_xor(y, off));
        }
        if ((threadIdx.x & 63) == 0) { wlo[w][l] = x; whi[w][l] = y; }
    }
    __syncthreads();
    if ((int)threadIdx.x < nx) {
        const int l = threadIdx.x;
        const double x = fmin(fmin(wlo[0][l], wlo[1][l]), fmin(wlo[2][l], wlo[3][l]));
        const double y = fmax(fmax(whi[0][l], whi[1][l]), fmax(whi[2][l], whi[3][l]));
        if (parts == 1) {
            P.s_lo[u * nx + l] = x;
            P.s_hi[u * nx + l] = y;
        } else {
            if (x < 0.0) atomic_grow(&P.s_lo[u * nx + l], x);
            if (y > 0.0) atomic_grow(&P.s_hi[u * nx + l], y);
        }
    }
}

static SmallArgs small_args(const leb_dynamics* dyn, int64_t units, const double* z, const double* v,
                            const double* mu, const double* sigma) {
    SmallArgs A;
    A.z = z; A.v = v; A.mu = mu; A.sigma = sigma; A.Q = dyn->coeffs;
    A.r_lo = A.r_hi = A.c_bar = A.rho_bar = nullptr;
    A.flags = nullptr; A.pad = 0.0;
    A.units = units; A.nx = dyn->nx; A.nu = dyn->nu; A.kind = dyn->kind;
    A.dt = dyn->dt; A.m = dyn->m;
    for (int i = 0; i < 3; ++i) A.J[i] = dyn->J[i];
    return A;
}

int launch_small_dyn(const leb_dynamics* dyn, int mode, int64_t units, const double* z, const double* v,
                     const double* mu, const double* sigma, double* r_lo, double* r_hi, double* c_bar,
                     double* rho_bar, double pad, uint32_t* flags, hipStream_t s) {
    SmallArgs A = small_args(dyn, units, z, v, mu, sigma);
    A.r_lo = r_lo; A.r_hi = r_hi; A.c_bar = c_bar; A.rho_bar = rho_bar; A.flags = flags; A.pad = pad;
    const dim3 b(256);
    if (dyn->kind == LEB_DYN_LINEAR || dyn->kind == LEB_DYN_QUADRATIC) {
        int G = 1;
        while (G < dyn->nx) G <<= 1;     // nx <= 64 for QUADRATIC
        if (dyn->kind == LEB_DYN_LINEAR) G = 1;
        const int64_t blocks = (units * G + 255) / 256;
        if (blocks > 0x7fffffff) return LEB_EINVAL;
        const dim3 g((unsigned)blocks);
        if (mode == LEB_IH_PATH) hipLaunchKernelGGL(small_poly_kernel<LEB_IH_PATH>, g, b, 0, s, A, G);
        else if (mode == LEB_IH_EXPAND) hipLaunchKernelGGL(small_poly_kernel<LEB_IH_EXPAND>, g, b, 0, s, A, G);
        else hipLaunchKernelGGL(small_poly_kernel<LEB_IH_CLASSIC>, g, b, 0, s, A, G);
    } else {
        const int rc = dyn->kind == LEB_DYN_QUAD3D      ? launch_small_entry<LEB_DYN_QUAD3D, 16>(mode, A, s)
                       : dyn->kind == LEB_DYN_SATELLITE ? launch_small_entry<LEB_DYN_SATELLITE, 4>(mode, A, s)
                       : dyn->nx == 2                   ? launch_small_entry<LEB_DYN_SINCOS, 4>(mode, A, s)
                                                        : launch_small_entry<LEB_DYN_SINCOS, 1>(mode, A, s);
        if (rc) return rc;
    }
    return hipGetLastError() == hipSuccess ? LEB_OK : LEB_EDEVICE;
}

}  // namespace leb

using namespace leb;

static int small_kind(const leb_dynamics* dyn) {
    return dyn->kind == LEB_DYN_LINEAR || dyn->kind == LEB_DYN_QUADRATIC || dyn->kind == LEB_DYN_SINCOS ||
           dyn->kind == LEB_DYN_SATELLITE || dyn->kind == LEB_DYN_QUAD3D;
}

extern "C" int leb_interval_hessian_bound(const leb_dynamics* dyn, int32_t mode, int32_t batch, int32_t N,
                                          const double* z, const double* v, const double* mu, const double* sigma,
                                          double* r_lo, double* r_hi, uint32_t* flags, void* stream) {
    int rc = check_dynamics(dyn);
    if (rc != LEB_OK) return rc;
    if (mode != LEB_IH_PATH && mode != LEB_IH_EXPAND && mode != LEB_IH_CLASSIC) return LEB_EINVAL;
    if (!small_kind(dyn)) return LEB_ENOTSUP;
    if (batch < 0 || N < 0) return LEB_EINVAL;
    const int64_t units = (int64_t)batch * N;
    if (units == 0) return LEB_OK;
    const int64_t nx = dyn->nx, nu = dyn->nu;
    if (!r_lo || !r_hi || (nx > 0 && !z) || (nu > 0 && !v) || !sigma) return LEB_EINVAL;
    const void* ptrs[] = {z, v, mu, sigma, r_lo, r_hi};
    for (const void* p : ptrs)
        if (p && !aligned8(p)) return LEB_EINVAL;
    if (flags && (reinterpret_cast<uintptr_t>(flags) & 3u)) return LEB_EINVAL;
    if (units * (nx + nu) > ((int64_t)1 << 46)) return LEB_EINVAL;
    return launch_small_dyn(dyn, mode, units, z, v, mu, sigma, r_lo, r_hi, nullptr, nullptr, 0.0, flags,
                            (hipStream_t)stream);
}

extern "C" int leb_sample_remainder(const leb_dynamics* dyn, int32_t batch, int32_t N, const double* z,
                                    const double* v, const double* mu, const double* sigma, int32_t K,
                                    const double* t, double* s_lo, double* s_hi, void* stream) {
    int rc = check_dynamics(dyn);
    if (rc != LEB_OK) return rc;
    if (!small_kind(dyn) || dyn->kind == LEB_DYN_LINEAR || dyn->nx + dyn->nu > SD_SAMPLE_N) return LEB_ENOTSUP;
    if (batch < 0 || N < 0 || K < 0) return LEB_EINVAL;
    const int64_t units = (int64_t)batch * N;
    if (units == 0) return LEB_OK;
    if (units > 0x7fffffff) return LEB_EINVAL;
    if (!z || (dyn->nu > 0 && !v) || !sigma || !s_lo || !s_hi || (K > 0 && !t)) return LEB_EINVAL;
    const void* ptrs[] = {z, v, mu, sigma, t, s_lo, s_hi};
    for (const void* p : ptrs)
        if (p && !aligned8(p)) return LEB_EINVAL;
    SampleArgs P;
    P.S = small_args(dyn, units, z, v, mu, sigma);
    P.t = t; P.K = K; P.s_lo = s_lo; P.s_hi = s_hi;
    // parts a unit: about four workgroups a compute unit in all (1,024), at least one
    // sample a thread; one part needs no clearing and no atomics
    const int64_t most = ((int64_t)K + 255) / 256;
    const int64_t want = units >= 512 ? 1 : 1024 / units;
    const int parts = (int)(most < 1 ? 1 : (want < most ? want : most));
    hipStream_t st = (hipStream_t)stream;
    if (parts > 1)
        hipLaunchKernelGGL(sample_zero_kernel, dim3((unsigned)((units * dyn->nx + 255) / 256)), dim3(256), 0, st, s_lo, s_hi,
                           units * dyn->nx);
    const dim3 g((unsigned)units, (unsigned)parts), b(256);
    switch (dyn->kind) {
    case LEB_DYN_SINCOS: hipLaunchKernelGGL(sample_rem_kernel<LEB_DYN_SINCOS>, g, b, 0, st, P, parts); break;
    case LEB_DYN_SATELLITE: hipLaunchKernelGGL(sample_rem_kernel<LEB_DYN_SATELLITE>, g, b, 0, st, P, parts); break;
    case LEB_DYN_QUAD3D: hipLaunchKernelGGL(sample_rem_kernel<LEB_DYN_QUAD3D>, g, b, 0, st, P, parts); break;
    default: hipLaunchKernelGGL(sample_rem_kernel<LEB_DYN_QUADRATIC>, g, b, 0, st, P, parts); break;
    }
    return hipGetLastError() == hipSuccess ? LEB_OK : LEB_EDEVICE;
}
