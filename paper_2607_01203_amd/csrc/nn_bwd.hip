// nn_bwd.hip -- adjoint of the ReLU-MLP remainder bound (sections IV.B and IV.D).
//
// The bound of nn.hip (CROWN with a full pass for every hidden layer's
// pre-activation bounds, Theorem 2 with J = J_g(a~)) is piecewise smooth in
// the nominal a~, the radii sigma and the offset mu; the paper differentiates
// it to shape the nominal trajectory.  This file computes, for
//     L = sum_rows g_hi r_hi + g_lo r_lo,
// dL/da~, dL/dsigma and dL/dmu of the exact-arithmetic bound (rounding
// allowances of the forward kernels are not part of it), by reverse mode.
//
// Forward quantities.  Box c = a~ + (dlo + dhi)/2, rho = (dhi - dlo)/2 with
// dlo = min(mu - sigma, 0), dhi = max(mu + sigma, 0).  Layer-1 bounds
// W_1 c + b_1 -/+ |W_1| rho.  The pass of target layer k (2 <= k <= L) runs
//     Lambda^(k-1) = rows of W_k,  for j = k-1 .. 1:
//       sel = (Lambda >= 0) for the upper pass, (Lambda < 0) for the lower one
//       Omega_j = Lambda^(j) (.) S_j,  S_j = sel ? s_j : a_j
//       beta += sum sel Lambda^(j) t_j + Omega_j b_j,  Lambda^(j-1) = Omega_j W_j
// with the relaxation s = u/(u-l), t = -s l, a = [u >= -l] of each unstable
// neuron (identity / zero for stable ones), and concretises
// Lambda^(0) c +/- |Lambda^(0)| rho + beta (k < L: bounds of layer k; k = L:
// Theorem 2 with Lambda^(0) - J in place of Lambda^(0)).
//
// Reverse.  With the row seeds y (g_hi / g_lo for k = L, the adjoints of the
// bounds u_k / l_k otherwise), the adjoint of one pass is
//     Lambda-bar^(0) = y (c +/- sign(D) rho),  c-bar += D^T y,  rho-bar +/-= |D|^T y
//     for j = 1 .. k-1:
//       Omega-bar_j = Lambda-bar^(j-1) W_j^T + y b_j^T
//       s-bar_j += sum_rows sel Omega-bar_j Lambda^(j),  t-bar_j += sum_rows sel y Lambda^(j)
//       Lambda-bar^(j) = Omega-bar_j (.) S_j + sel y t_j      (j < k-1)
// (D = Lambda^(0) - J for k = L, Lambda^(0) otherwise), and the relaxation
// adjoint of an unstable neuron is
//     u-bar = (-l s-bar + l^2 t-bar) / (u-l)^2,  l-bar = (u s-bar - u^2 t-bar) / (u-l)^2.
// Passes run from k = L down to 2: the bounds of layer j receive adjoints
// only from passes with k > j, so each layer's adjoint is complete when its
// own pass is reversed.  J a~ - g(a~) has derivative 0 (J is locally constant).
//
// GPU design.  Sums are taken in a fixed order and later passes add to the per-neuron
// sums in launch order, so the result is deterministic.  Three forms:
//  * 16 inputs, at most three hidden layers (the usual case): the forward passes are the
//    bound's kernels (nn_hid.hpp), storing the levels of unstable target rows, the only
//    ones read back; the reverse passes keep the chain in registers (nn_rev_kernel).
//  * other inputs, at most three hidden layers: one workgroup of 256 lanes per (box, pass
//    direction), 16-row blocks on FP64 MFMA; lane q owns neuron column q of every level,
//    applies the relaxation selection to it and keeps its sums; every pass has a forward
//    launch that stores its levels and a reverse launch that reads them back; products
//    run over the neurons that are not stably inactive (see the MFMA section below).
//  * deeper networks, on the VALU: 8-row blocks, Lambda^(j) of the lane's column kept in
//    registers for the reverse sweep; hidden-layer passes store their levels, the output
//    pass recomputes its chain; narrow outputs (the input layer) split the sum over lane
//    slices added in a fixed order.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>
#include <vector>

#include "dpp.hpp"
#include "leb.h"
#include "leb_internal.hpp"
#include "nn_hid.hpp"
#include "nn_net.hpp"

namespace leb {

constexpr int NB_R = 8;          // target rows per block
constexpr int NB_T = 256;        // lanes per workgroup
constexpr int NB_CHUNK = 4096;   // most boxes per chunk of the workspace
constexpr int NB_CHUNK_MIN = 32; // fewest (deep, wide networks)
constexpr size_t NB_LV_BUDGET = (size_t)8 << 30;   // workspace bytes that set the chunk size

struct NbArgs {
    int L;
    int w[NN_MAXL + 1];
    const double* W[NN_MAXL];
    const double* WT[NN_MAXL];
    const double* b[NN_MAXL];
    int nx, nu;
    int k;                         // target layer of a pass; layer of a relaxation adjoint
    int64_t u0;                    // first unit of the chunk
    const double* z; const double* v; const double* mu; const double* sigma;
    const double* g_lo; const double* g_hi;
    double* gz; double* gv; double* gmu; double* gsigma;
    // chunk workspace (box-major)
    double* cr;                    // [box][2][NN_MAXW]          c, rho
    double* zn;                    // [box][NN_MAXL][NN_MAXW]    nominal pre-activations of hidden layer j (index j-1)
    double* bd;                    // [box][NN_MAXL][2][NN_MAXW] lo, hi of hidden layer j
    double* st;                    // [box][2][NN_MAXL][2][NN_MAXW] s-bar, t-bar per pass direction
    double* ub;                    // [box][NN_MAXL][2][NN_MAXW] u-bar, l-bar of hidden layer j
    double* cg;                    // [box][2][2][NN_MAXW]       c-bar, rho-bar per pass direction
    uint32_t* ok;                  // [box] 1: valid input
    double* jac;                   // 16 inputs: [box][w[L]][16] the Jacobian's rows
    double* lv;                    // [box][2][lv_bm] levels Lambda^(j) of the hidden-layer passes
    size_t lv_bm;                  // doubles per (box, direction)
    int lv_off[NN_MAXL][NN_MAXL];  // offset of level j of pass k: [row][column], w[k] x w[j]
};

__device__ __forceinline__ size_t ix_cr(int box, int which) { return ((size_t)box * 2 + which) * NN_MAXW; }
__device__ __forceinline__ size_t ix_zn(int box, int j) { return ((size_t)box * NN_MAXL + j - 1) * NN_MAXW; }
__device__ __forceinline__ size_t ix_bd(int box, int j, int hi) {
    return (((size_t)box * NN_MAXL + j - 1) * 2 + hi) * NN_MAXW;
}
__device__ __forceinline__ size_t ix_st(int box, int mode, int j, int which) {
    return ((((size_t)box * 2 + mode) * NN_MAXL + j - 1) * 2 + which) * NN_MAXW;
}
__device__ __forceinline__ size_t ix_ub(int box, int j, int which) {
    return (((size_t)box * NN_MAXL + j - 1) * 2 + which) * NN_MAXW;
}
__device__ __forceinline__ size_t ix_cg(int box, int mode, int which) {
    return (((size_t)box * 2 + mode) * 2 + which) * NN_MAXW;
}

// out[r][i] = sum_{p < len} X[p][r] M[p nc + i] for i < nc, X in LDS as [p][NB_R];
// lane q < nc receives column q.  Narrow outputs split p over 256 / nc lane
// slices, added in slice order.  Every lane must call it (it may hold a barrier).
__device__ __forceinline__ void nb_rowmat(const double* __restrict__ M, int nc, int len, const double* sX,
                                          double* sP, int q, double acc[NB_R]) {
    const int S = nc >= NB_T ? 1 : NB_T / nc;
    const int i = q % nc, sl = q / nc;
#pragma unroll
    for (int r = 0; r < NB_R; ++r) acc[r] = 0.0;
    if (sl < S) {
        const int p0 = (int)(((int64_t)sl * len) / S), p1 = (int)(((int64_t)(sl + 1) * len) / S);
        const double* Mi = M + i;
#pragma unroll 4
        for (int p = p0; p < p1; ++p) {
            const double w = Mi[(size_t)p * nc];
            const double* x = sX + p * NB_R;
#pragma unroll
            for (int r = 0; r < NB_R; ++r) acc[r] = __builtin_fma(x[r], w, acc[r]);
        }
    }
    if (S > 1) {
        if (sl >= 1 && sl < S) {
#pragma unroll
            for (int r = 0; r < NB_R; ++r) sP[((sl - 1) * nc + i) * NB_R + r] = acc[r];
        }
        lds_barrier();
        if (q < nc) {
            for (int s2 = 1; s2 < S; ++s2) {
#pragma unroll
                for (int r = 0; r < NB_R; ++r) acc[r] += sP[((s2 - 1) * nc + q) * NB_R + r];
            }
        }
    }
}

// per box: validity, the box (c, rho), nominal pre-activations, layer-1
// bounds, and zeroed adjoint sums
__global__ void __launch_bounds__(NB_T) nb_box_kernel(NbArgs A) {
    __shared__ double s_a[NN_MAXW], s_c[NN_MAXW], s_r[NN_MAXW];
    __shared__ uint32_t s_bad;
    const int box = blockIdx.x, q = threadIdx.x;
    const int64_t unit = A.u0 + box;
    const int n0 = A.w[0], L = A.L;
    if (q == 0) s_bad = 0;
    __syncthreads();
    if (q < n0) {
        const double x = q < A.nx ? A.z[unit * A.nx + q] : A.v[unit * A.nu + (q - A.nx)];
        const double sg = A.sigma[unit * n0 + q];
        const double mu = A.mu ? A.mu[unit * n0 + q] : 0.0;
        if (!isfinite(x) || !isfinite(sg) || !isfinite(mu) || !(sg >= 0.0)) atomicOr(&s_bad, 1u);
        const double dlo = fmin(mu - sg, 0.0), dhi = fmax(mu + sg, 0.0);
        s_a[q] = x;
        s_c[q] = x + 0.5 * (dlo + dhi);
        s_r[q] = 0.5 * (dhi - dlo);
        A.cr[ix_cr(box, 0) + q] = s_c[q];
        A.cr[ix_cr(box, 1) + q] = s_r[q];
    }
    // zero the adjoint sums of this box
    for (int j = 1; j < L; ++j)
        for (int md = 0; md < 2; ++md)
            for (int wh = 0; wh < 2; ++wh) A.st[ix_st(box, md, j, wh) + q] = 0.0;
    for (int md = 0; md < 2; ++md)
        for (int wh = 0; wh < 2; ++wh) A.cg[ix_cg(box, md, wh) + q] = 0.0;
    __syncthreads();
    if (q == 0) A.ok[box] = s_bad ? 0u : 1u;
    const int n1 = A.w[1];
    if (q < n1) {
        const double* Wr = A.W[0] + (size_t)q * n0;
        double lin = A.b[0][q], mag = 0.0;
        for (int p = 0; p < n0; ++p) {
            lin = __builtin_fma(Wr[p], s_c[p], lin);
            mag = __builtin_fma(fabs(Wr[p]), s_r[p], mag);
        }
        A.bd[ix_bd(box, 1, 0) + q] = lin - mag;
        A.bd[ix_bd(box, 1, 1) + q] = lin + mag;
    }
    // nominal pre-activations of the hidden layers (the masks of J)
    for (int l = 0; l < L - 1; ++l) {
        const int in = A.w[l], out = A.w[l + 1];
        double zz = 0.0;
        if (q < out) {
            zz = A.b[l][q];
            const double* WT = A.WT[l];
            for (int p = 0; p < in; ++p) zz = __builtin_fma(WT[(size_t)p * out + q], s_a[p], zz);
        }
        __syncthreads();
        if (q < out) {
            A.zn[ix_zn(box, l + 1) + q] = zz;
            s_a[q] = zz > 0.0 ? zz : 0.0;
        }
        __syncthreads();
    }
}

// nb_box_kernel for 16 boxes a workgroup (nn_hid.hpp: group_products; bitwise the same sums):
// 3,200 boxes of 16-256-256-256-12 57 us (one box a workgroup 225 us).
constexpr size_t NBG_LDS = (size_t)2 * NN_MAXW * NNG_RS * sizeof(double);

__global__ void __launch_bounds__(NNG_T) nb_box_group_kernel(NbArgs A, int nact) {
    extern __shared__ __attribute__((aligned(16))) double X[];       // [2][NN_MAXW][NNG_RS]
    __shared__ uint32_t s_bad[NNG_BOXES];
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = blockIdx.x * NNG_BOXES, nb = min(NNG_BOXES, nact - b0);
    const int n0 = A.w[0], n1 = A.w[1], L = A.L;
    auto X_ = [&](int c, int n, int b) -> double& { return X[(c * NN_MAXW + n) * NNG_RS + b]; };
    if (tid < NNG_BOXES) s_bad[tid] = 0;
    __syncthreads();
    auto nominal = [&](int b, int q) {
        const int64_t unit = A.u0 + b0 + min(b, nb - 1);
        return q < A.nx ? A.z[unit * A.nx + q] : A.v[unit * A.nu + (q - A.nx)];
    };
    for (int e = tid; e < NNG_BOXES * n0; e += NNG_T) {
        const int b = e / n0, q = e - b * n0, box = b0 + min(b, nb - 1);
        const double x = nominal(b, q);
        const double sg = A.sigma[(A.u0 + box) * n0 + q];
        const double mu = A.mu ? A.mu[(A.u0 + box) * n0 + q] : 0.0;
        if (!isfinite(x) || !isfinite(sg) || !isfinite(mu) || !(sg >= 0.0)) atomicOr(&s_bad[b], 1u);
        const double dlo = fmin(mu - sg, 0.0), dhi = fmax(mu + sg, 0.0);
        const double c = x + 0.5 * (dlo + dhi), h = 0.5 * (dhi - dlo);
        X_(0, q, b) = c;
        X_(1, q, b) = h;
        if (b < nb) { A.cr[ix_cr(box, 0) + q] = c; A.cr[ix_cr(box, 1) + q] = h; }
    }
    // zero the adjoint sums of these boxes
    for (int b = 0; b < nb; ++b) {
        const int half = tid >> 8, q = tid & 255;
        for (int j = 1; j < L; ++j)
            for (int wh = 0; wh < 2; ++wh) A.st[ix_st(b0 + b, half, j, wh) + q] = 0.0;
        for (int wh = 0; wh < 2; ++wh) A.cg[ix_cg(b0 + b, half, wh) + q] = 0.0;
    }
    __syncthreads();
    if (tid < nb) A.ok[b0 + tid] = s_bad[tid] ? 0u : 1u;
    // layer-1 bounds
    {
        d4 acc[2][2];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = 16 * (wave + 8 * q) + 4 * i + g;
                acc[q][0][i] = n < n1 ? A.b[0][n] : 0.0;
                acc[q][1][i] = 0.0;
            }
        group_products<2, true, false>(A.WT[0], n0, n1, X, wave, r, g, acc);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (16 * (wave + 8 * q) >= n1) break;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = 16 * (wave + 8 * q) + 4 * i + g;
                X_(0, n, r) = acc[q][0][i] - acc[q][1][i];
                X_(1, n, r) = acc[q][0][i] + acc[q][1][i];
            }
        }
        __syncthreads();
        for (int e = tid; e < nb * n1; e += NNG_T) {
            const int b = e / n1, n = e - b * n1;
            A.bd[ix_bd(b0 + b, 1, 0) + n] = X_(0, n, b);
            A.bd[ix_bd(b0 + b, 1, 1) + n] = X_(1, n, b);
        }
        __syncthreads();
    }
    // nominal pre-activations of the hidden layers (the masks of J)
    for (int e = tid; e < NNG_BOXES * n0; e += NNG_T) X_(0, e % n0, e / n0) = nominal(e / n0, e % n0);
    __syncthreads();
    for (int l = 0; l < L - 1; ++l) {
        const int out = A.w[l + 1];
        d4 acc[2][1];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = 16 * (wave + 8 * q) + 4 * i + g;
                acc[q][0][i] = n < out ? A.b[l][n] : 0.0;
            }
        if (l == 0) group_products<1, true, false>(A.WT[l], A.w[l], out, X, wave, r, g, acc);
        else group_products<1, true, true>(A.WT[l], A.w[l], out, X, wave, r, g, acc);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (16 * (wave + 8 * q) >= out) break;
#pragma unroll
            for (int i = 0; i < 4; ++i) X_(0, 16 * (wave + 8 * q) + 4 * i + g, r) = acc[q][0][i];
        }
        __syncthreads();
        for (int e = tid; e < nb * out; e += NNG_T) {
            const int b = e / out, n = e - b * out;
            A.zn[ix_zn(b0 + b, l + 1) + n] = X_(0, n, b);
        }
    }
}

// One CROWN pass of target layer A.k for one box (blockIdx.x) and direction
// (blockIdx.y: 0 upper, 1 lower).  REV = false: the bounds of layer k
// (hi for the upper pass, lo for the lower one).  REV = true: the adjoint of
// the pass, added to the per-neuron sums.  LV >= k - 1: levels kept per lane.
template <bool REV, int LV>
__global__ void __launch_bounds__(NB_T) nb_pass_kernel(NbArgs A) {
    __shared__ __attribute__((aligned(16))) double sX[NN_MAXW * NB_R];
    __shared__ __attribute__((aligned(16))) double sP[NN_MAXW * NB_R];
    __shared__ double sRed[NB_T / 64][NB_R];
    const int box = blockIdx.x, mode = blockIdx.y, q = threadIdx.x;
    if (!A.ok[box]) return;
    const bool upper = mode == 0;
    const double sgn = upper ? 1.0 : -1.0;
    const int k = A.k, L = A.L, n0 = A.w[0];
    const int rows = A.w[k], nk1 = A.w[k - 1];
    const double* Wk = A.W[k - 1];
    const double cq = q < n0 ? A.cr[ix_cr(box, 0) + q] : 0.0;
    const double rq = q < n0 ? A.cr[ix_cr(box, 1) + q] : 0.0;
    double sacc[LV], tacc[LV];
#pragma unroll
    for (int j = 0; j < LV; ++j) { sacc[j] = 0.0; tacc[j] = 0.0; }
    double cacc = 0.0, racc = 0.0;

    for (int r0 = 0; r0 < rows; r0 += NB_R) {
        const int nr = min(NB_R, rows - r0);
        double lam[LV][NB_R];                   // Lambda^(j) of column q, j = 0 .. k-2
        double bpart[NB_R];
#pragma unroll
        for (int r = 0; r < NB_R; ++r) bpart[r] = 0.0;
        double* lvb = A.lv + ((size_t)box * 2 + mode) * A.lv_bm;
        if (REV && k < L) {
            // the levels stored by this layer's forward pass
#pragma unroll
            for (int j = 0; j < LV; ++j) {
                if (j > k - 2 || q >= A.w[j]) continue;
                const double* src = lvb + A.lv_off[k][j] + (size_t)r0 * A.w[j] + q;
#pragma unroll
                for (int r = 0; r < NB_R; ++r) lam[j][r] = r < nr ? src[(size_t)r * A.w[j]] : 0.0;
            }
        }
        // ---- forward chain of the block, j = k-1 .. 1 (every pass but the
        // reverse of a hidden layer's)
#pragma unroll
        for (int j = LV; j >= 1; --j) {
            if (j > k - 1 || (REV && k < L)) continue;
            const int nj = A.w[j];
            if (q < nj) {
                double s, t, a;
                nb_relax(A.bd[ix_bd(box, j, 0) + q], A.bd[ix_bd(box, j, 1) + q], s, t, a);
                const double bj = A.b[j - 1][q];
#pragma unroll
                for (int r = 0; r < NB_R; ++r) {
                    double lm;
                    if (j == k - 1) lm = r < nr ? Wk[(size_t)(r0 + r) * nk1 + q] : 0.0;
                    else lm = lam[j < LV ? j : 0][r];     // j < LV whenever j < k - 1
                    const bool sel = upper ? lm >= 0.0 : lm < 0.0;
                    const double om = lm * (sel ? s : a);
                    if (!REV) bpart[r] += (sel ? lm * t : 0.0) + om * bj;
                    sX[q * NB_R + r] = om;
                }
            }
            lds_barrier();
            double acc[NB_R];
            nb_rowmat(A.W[j - 1], A.w[j - 1], nj, sX, sP, q, acc);
            if (q < A.w[j - 1]) {
#pragma unroll
                for (int r = 0; r < NB_R; ++r) lam[j - 1][r] = acc[r];
                if (!REV) {
                    double* dst = lvb + A.lv_off[k][j - 1] + (size_t)r0 * A.w[j - 1] + q;
#pragma unroll
                    for (int r = 0; r < NB_R; ++r)
                        if (r < nr) dst[(size_t)r * A.w[j - 1]] = acc[r];
                }
            }
            lds_barrier();
        }
        if (!REV) {
            // concretise: row value = b_k + beta parts + Lambda^(0) c +/- |Lambda^(0)| rho
            if (q < n0) {
#pragma unroll
                for (int r = 0; r < NB_R; ++r) bpart[r] += lam[0][r] * cq + sgn * fabs(lam[0][r]) * rq;
            }
            const int wv = q >> 6;
#pragma unroll
            for (int r = 0; r < NB_R; ++r) {
                double x = bpart[r];
#pragma unroll
                for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
                if ((q & 63) == 0) sRed[wv][r] = x;
            }
            lds_barrier();
            if (q < nr) {
                double x = A.b[k - 1][r0 + q];
                for (int w2 = 0; w2 < NB_T / 64; ++w2) x += sRed[w2][q];
                A.bd[ix_bd(box, k, upper ? 1 : 0) + r0 + q] = x;
            }
            lds_barrier();
            continue;
        }
        // ---- reverse sweep of the block
        double y[NB_R];
#pragma unroll
        for (int r = 0; r < NB_R; ++r) {
            double yy = 0.0;
            if (r < nr) {
                if (k == L) yy = (upper ? A.g_hi : A.g_lo)[(A.u0 + box) * rows + r0 + r];
                else yy = A.ub[ix_ub(box, k, upper ? 0 : 1) + r0 + r];
            }
            y[r] = yy;
        }
        double jv[NB_R];
#pragma unroll
        for (int r = 0; r < NB_R; ++r) jv[r] = 0.0;
        if (k == L) {
            // the rows of J = W_L D_{L-1} W_{L-1} ... D_1 W_1 (D = [z^ > 0]) for this block
#pragma unroll
            for (int r = 0; r < NB_R; ++r) jv[r] = (q < nk1 && r < nr) ? Wk[(size_t)(r0 + r) * nk1 + q] : 0.0;
            for (int j = L - 1; j >= 1; --j) {
                const int nj = A.w[j];
                if (q < nj) {
                    const double on = A.zn[ix_zn(box, j) + q] > 0.0 ? 1.0 : 0.0;
#pragma unroll
                    for (int r = 0; r < NB_R; ++r) sX[q * NB_R + r] = jv[r] * on;
                }
                lds_barrier();
                nb_rowmat(A.W[j - 1], A.w[j - 1], nj, sX, sP, q, jv);
                lds_barrier();
            }
        }
        // seeds of Lambda^(0) and the direct c / rho terms
        if (q < n0) {
#pragma unroll
            for (int r = 0; r < NB_R; ++r) {
                const double d = lam[0][r] - jv[r];
                const double sd = d > 0.0 ? 1.0 : (d < 0.0 ? -1.0 : 0.0);
                cacc += y[r] * d;
                racc += sgn * y[r] * fabs(d);
                sX[q * NB_R + r] = y[r] * (cq + sgn * sd * rq);
            }
        }
        lds_barrier();
#pragma unroll
        for (int j = 1; j <= LV; ++j) {
            if (j > k - 1) continue;
            const int nj = A.w[j];
            double ob[NB_R];
            nb_rowmat(A.WT[j - 1], nj, A.w[j - 1], sX, sP, q, ob);
            lds_barrier();                      // sX is rewritten below
            if (q < nj) {
                double s, t, a;
                nb_relax(A.bd[ix_bd(box, j, 0) + q], A.bd[ix_bd(box, j, 1) + q], s, t, a);
                const double bj = A.b[j - 1][q];
                double sa = 0.0, ta = 0.0;
#pragma unroll
                for (int r = 0; r < NB_R; ++r) {
                    double lm;
                    if (j == k - 1) lm = r < nr ? Wk[(size_t)(r0 + r) * nk1 + q] : 0.0;
                    else lm = lam[j < LV ? j : 0][r];     // j < LV whenever j < k - 1
                    const bool sel = upper ? lm >= 0.0 : lm < 0.0;
                    const double obr = ob[r] + y[r] * bj;
                    if (sel) {
                        sa += obr * lm;
                        ta += y[r] * lm;
                    }
                    if (j < k - 1) sX[q * NB_R + r] = obr * (sel ? s : a) + (sel ? y[r] * t : 0.0);
                }
                sacc[j - 1] += sa;
                tacc[j - 1] += ta;
            }
            lds_barrier();
        }
    }
    if (REV) {
#pragma unroll
        for (int j = 1; j <= LV; ++j) {
            if (j > k - 1) continue;
            if (q < A.w[j]) {
                A.st[ix_st(box, mode, j, 0) + q] += sacc[j - 1];
                A.st[ix_st(box, mode, j, 1) + q] += tacc[j - 1];
            }
        }
        if (q < n0) {
            A.cg[ix_cg(box, mode, 0) + q] += cacc;
            A.cg[ix_cg(box, mode, 1) + q] += racc;
        }
    }
}

// ---------------------------------------------------------------- MFMA form
//
// Networks with at most three hidden layers: the row-block products run on
// FP64 MFMA (v_mfma_f64_16x16x4f64) with 16-row blocks.  The operand (16 rows
// x len) and the product (16 rows x nc) sit in LDS as [neuron][row] with a
// row stride of 17 doubles, so the A-operand reads (lane l: row l % 16 of
// k-step 4 kk + l / 16) are consecutive and the owner lanes' column reads
// spread over the banks.  B operands (the weights) come from L2, one per lane
// and tile per k-step, the next k-step's loaded before this one's MFMAs.
// Every pass, the output pass included, has a forward launch that stores its
// levels; the reverse launches read them back, so no level lives in
// registers across a product.
typedef double nbd4 __attribute__((ext_vector_type(4)));
constexpr int NBM_R = 16;        // rows per block
constexpr int NBM_RS = 17;       // LDS row stride of operand and product

// sD[col][row] = sum_{p < len} sA[p][row] M[kl[p] ld + cl[col]], col < nc,
// 16 rows; kl = NULL: kl[p] = p, cl = NULL: cl[c] = c.  len a multiple of 4
// (possibly 0), nc of 16.  Every lane calls it; it ends with a barrier after
// which sD is complete (and sA no longer read).
__device__ __forceinline__ void nbm_mm(const double* __restrict__ M, int ld, int nc, int len, const int* kl,
                                       const int* cl, const double* sA, double* sD, int q) {
    const int w = q >> 6, l = q & 63, lr = l & 15, lq = l >> 4;
    const int nt = nc >> 4, nk = len >> 2;
    auto krow = [&](int p) { return (size_t)(kl ? kl[p] : p) * ld; };
    auto kcol = [&](int t) { return (size_t)(cl ? cl[16 * t + lr] : 16 * t + lr); };
    if (nt >= 4) {
        // column tiles t = w, w + 4, ... of this wave over the whole k range
        nbd4 acc[4];
#pragma unroll
        for (int s2 = 0; s2 < 4; ++s2) acc[s2] = nbd4{0.0, 0.0, 0.0, 0.0};
        double bn[4];
#pragma unroll
        for (int s2 = 0; s2 < 4; ++s2) {
            const int t = w + 4 * s2;
            bn[s2] = (t < nt && nk > 0) ? M[krow(lq) + kcol(t)] : 0.0;
        }
        for (int kk = 0; kk < nk; ++kk) {
            double b[4];
#pragma unroll
            for (int s2 = 0; s2 < 4; ++s2) b[s2] = bn[s2];
            if (kk + 1 < nk) {
#pragma unroll
                for (int s2 = 0; s2 < 4; ++s2) {
                    const int t = w + 4 * s2;
                    bn[s2] = t < nt ? M[krow(4 * kk + 4 + lq) + kcol(t)] : 0.0;
                }
            }
            const double av = sA[(4 * kk + lq) * NBM_RS + lr];
#pragma unroll
            for (int s2 = 0; s2 < 4; ++s2)
                if (w + 4 * s2 < nt) acc[s2] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, b[s2], acc[s2], 0, 0, 0);
        }
#pragma unroll
        for (int s2 = 0; s2 < 4; ++s2) {
            const int t = w + 4 * s2;
            if (t < nt) {
#pragma unroll
                for (int i = 0; i < 4; ++i) sD[(16 * t + lr) * NBM_RS + 4 * i + lq] = acc[s2][i];
            }
        }
        lds_barrier();
        return;
    }
    // narrow output (1 to 3 tiles): the k range in four quarters, one per
    // wave, partials added in wave order
    // two k-steps per trip into two accumulators (their loads issued
    // together, two independent MFMA chains), added at the end
    nbd4 acc[3], acc2[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) { acc[t] = nbd4{0.0, 0.0, 0.0, 0.0}; acc2[t] = nbd4{0.0, 0.0, 0.0, 0.0}; }
    const int k0 = (w * nk) >> 2, k1 = ((w + 1) * nk) >> 2;
    int kk = k0;
    for (; kk + 1 < k1; kk += 2) {
        const double av0 = sA[(4 * kk + lq) * NBM_RS + lr];
        const double av1 = sA[(4 * kk + 4 + lq) * NBM_RS + lr];
        double b0[3], b1[3];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            b0[t] = t < nt ? M[krow(4 * kk + lq) + kcol(t)] : 0.0;
            b1[t] = t < nt ? M[krow(4 * kk + 4 + lq) + kcol(t)] : 0.0;
        }
#pragma unroll
        for (int t = 0; t < 3; ++t)
            if (t < nt) {
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av0, b0[t], acc[t], 0, 0, 0);
                acc2[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av1, b1[t], acc2[t], 0, 0, 0);
            }
    }
    if (kk < k1) {
        const double av = sA[(4 * kk + lq) * NBM_RS + lr];
#pragma unroll
        for (int t = 0; t < 3; ++t)
            if (t < nt) {
                const double bv = M[krow(4 * kk + lq) + kcol(t)];
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[t], 0, 0, 0);
            }
    }
#pragma unroll
    for (int t = 0; t < 3; ++t) acc[t] += acc2[t];
    double* part = sD + 1024;            // [wave][tile][i][lane], past the product's 3 tiles
#pragma unroll
    for (int t = 0; t < 3; ++t)
        if (t < nt) {
#pragma unroll
            for (int i = 0; i < 4; ++i) part[((w * 3 + t) * 4 + i) * 64 + l] = acc[t][i];
        }
    lds_barrier();
    for (int e = q; e < nc * NBM_R; e += NB_T) {
        const int col = e >> 4, row = e & 15;
        const int t = col >> 4, li = (row & 3) * 16 + (col & 15), i = row >> 2;
        double x = 0.0;
        for (int w2 = 0; w2 < 4; ++w2) x += part[((w2 * 3 + t) * 4 + i) * 64 + li];
        sD[col * NBM_RS + row] = x;
    }
    lds_barrier();
}

// zero the operand rows tot .. len-1 (the padding of a neuron list)
__device__ __forceinline__ void nbm_pad(double* sA, int tot, int len, int q) {
    for (int e = q; e < (len - tot) * NBM_R; e += NB_T) sA[(tot + e / NBM_R) * NBM_RS + e % NBM_R] = 0.0;
}

// One CROWN pass of target layer A.k (2 <= k <= L) for one box and direction,
// MFMA form.  FWD: the levels of every 16-row block into lv, and for a
// hidden layer its bounds.  REV: the adjoint of the pass from the stored levels.
template <bool REV>
__global__ void __launch_bounds__(NB_T) __attribute__((amdgpu_waves_per_eu(2))) nbm_pass_kernel(NbArgs A) {
    __shared__ __attribute__((aligned(16))) double sA[NN_MAXW * NBM_RS];
    __shared__ __attribute__((aligned(16))) double sD[NN_MAXW * NBM_RS];
    // per hidden layer j (index j-1): the neurons that are not stably inactive
    // (an inactive neuron's column of Omega, and of Lambda-bar, is exactly 0,
    // and its own columns of Lambda and Omega-bar are never used), padded with
    // entry 0 to a multiple of 4 (k range) and of 16 (output columns); pos: a
    // neuron's place in the list.  Products over a hidden layer's neurons, in
    // k or in output columns, run over its list; their outputs sit at list
    // positions.  In a reverse launch the last layer (j = k - 1) lists its unstable
    // neurons only: nothing is propagated past it, and s-bar and t-bar are used
    // nowhere else (pass of layer 3 over 3,200 boxes of 16-256-256-256-12: 1.56 ms with
    // every active neuron's columns, 1.10 ms without).
    __shared__ int sList[3][NN_MAXW], sPos[3][NN_MAXW], sLen[3], sLen16[3], sTot[3];
    __shared__ int sCnt[NB_T / 64];
    // reverse launches: the target rows that are run.  A hidden layer's adjoint is
    // exactly 0 in its stable neurons (their relaxation does not depend on the
    // bounds), so its pass runs over the others only: layers 2 and 3 of the
    // 16-256-256-256-12 network have 16 and 22 % unstable neurons, and their
    // passes over 3,200 boxes take 0.38 and 1.10 ms (over every row: 1.38, 5.82).
    __shared__ int sRow[NN_MAXW];
    const int box = blockIdx.x, mode = blockIdx.y, q = threadIdx.x;
    if (!A.ok[box]) return;
    int rows = A.w[A.k];
    if (REV) {
        const bool keep = q < rows && (A.k == A.L || !(A.ub[ix_ub(box, A.k, mode) + q] == 0.0));
        const uint64_t bal = __ballot(keep);
        if ((q & 63) == 0) sCnt[q >> 6] = __popcll(bal);
        lds_barrier();
        int off = 0, tot = 0;
        for (int w2 = 0; w2 < NB_T / 64; ++w2) {
            if (w2 < (q >> 6)) off += sCnt[w2];
            tot += sCnt[w2];
        }
        if (keep) sRow[off + __popcll(bal & ((1ull << (q & 63)) - 1ull))] = q;
        rows = tot;
        lds_barrier();
        if (rows == 0) return;
    }
    for (int j = 1; j <= A.k - 1; ++j) {
        const int nj = A.w[j];
        const double lo = q < nj ? A.bd[ix_bd(box, j, 0) + q] : -1.0, hi = q < nj ? A.bd[ix_bd(box, j, 1) + q] : -1.0;
        const bool keep = REV && j == A.k - 1 ? lo < 0.0 && hi > 0.0 : lo >= 0.0 || hi > 0.0;
        const uint64_t bal = __ballot(keep);
        if ((q & 63) == 0) sCnt[q >> 6] = __popcll(bal);
        lds_barrier();
        int off = 0, tot = 0;
        for (int w2 = 0; w2 < NB_T / 64; ++w2) {
            if (w2 < (q >> 6)) off += sCnt[w2];
            tot += sCnt[w2];
        }
        const int pos = off + __popcll(bal & ((1ull << (q & 63)) - 1ull));
        if (keep) sList[j - 1][pos] = q;
        if (q < nj) sPos[j - 1][q] = keep ? pos : -1;
        const int padded = (tot + 3) & ~3, padded16 = (tot + 15) & ~15;
        if (q >= tot && q < padded16) sList[j - 1][q] = 0;
        if (q == 0) { sLen[j - 1] = padded; sLen16[j - 1] = padded16; sTot[j - 1] = tot; }
        lds_barrier();
    }
    const bool upper = mode == 0;
    const double sgn = upper ? 1.0 : -1.0;
    const int k = A.k, L = A.L, n0 = A.w[0];
    const int nk1 = A.w[k - 1], rows_k = A.w[k];
    const double* Wk = A.W[k - 1];
    const double cq = q < n0 ? A.cr[ix_cr(box, 0) + q] : 0.0;
    const double rq = q < n0 ? A.cr[ix_cr(box, 1) + q] : 0.0;
    double* lvb = A.lv + ((size_t)box * 2 + mode) * A.lv_bm;
    double sacc[3] = {0.0, 0.0, 0.0}, tacc[3] = {0.0, 0.0, 0.0};
    double cacc = 0.0, racc = 0.0;
    // forward launches: the relaxation and bias of the lane's neuron in each
    // layer j < k (loaded once), and the rows of W_k of the next block (loaded
    // while the current block computes)
    double fs[3] = {0.0, 0.0, 0.0}, ft[3] = {0.0, 0.0, 0.0}, fa[3] = {0.0, 0.0, 0.0}, fb[3] = {0.0, 0.0, 0.0};
    double wk[NBM_R];
    // reverse launches: Lambda^(0) rows of the block (lanes q < n0), loaded a block ahead
    double l0n[NBM_R];
    if (REV) {
#pragma unroll
        for (int r = 0; r < NBM_R; ++r)
            l0n[r] = (q < n0 && r < rows) ? lvb[A.lv_off[k][0] + (size_t)sRow[r] * n0 + q] : 0.0;
    }
    if (!REV) {
#pragma unroll
        for (int j = 1; j <= 3; ++j) {
            if (j <= k - 1 && q < A.w[j]) {
                nb_relax(A.bd[ix_bd(box, j, 0) + q], A.bd[ix_bd(box, j, 1) + q], fs[j - 1], ft[j - 1], fa[j - 1]);
                fb[j - 1] = A.b[j - 1][q];
            }
        }
#pragma unroll
        for (int r = 0; r < NBM_R; ++r) wk[r] = (q < nk1 && r < rows) ? Wk[(size_t)r * nk1 + q] : 0.0;
    }

    for (int r0 = 0; r0 < rows; r0 += NBM_R) {
        const int nr = min(NBM_R, rows - r0);
        if (!REV) {
            double bpart[NBM_R];
#pragma unroll
            for (int r = 0; r < NBM_R; ++r) bpart[r] = 0.0;
            for (int j = k - 1; j >= 1; --j) {
                const int nj = A.w[j];
                const int pq = q < nj ? sPos[j - 1][q] : -1;
                if (pq >= 0) {
                    const double s = j == 1 ? fs[0] : (j == 2 ? fs[1] : fs[2]);
                    const double t = j == 1 ? ft[0] : (j == 2 ? ft[1] : ft[2]);
                    const double a = j == 1 ? fa[0] : (j == 2 ? fa[1] : fa[2]);
                    const double bj = j == 1 ? fb[0] : (j == 2 ? fb[1] : fb[2]);
#pragma unroll
                    for (int r = 0; r < NBM_R; ++r) {
                        const double lm = j == k - 1 ? wk[r] : sD[pq * NBM_RS + r];
                        const bool sel = upper ? lm >= 0.0 : lm < 0.0;
                        const double om = lm * (sel ? s : a);
                        bpart[r] += (sel ? lm * t : 0.0) + om * bj;
                        sA[pq * NBM_RS + r] = om;
                    }
                }
                if (j == k - 1) {
                    // the next block's rows of W_k
                    const int r1 = r0 + NBM_R;
#pragma unroll
                    for (int r = 0; r < NBM_R; ++r)
                        wk[r] = (q < nk1 && r1 + r < rows) ? Wk[(size_t)(r1 + r) * nk1 + q] : 0.0;
                }
                const int len = sLen[j - 1];
                nbm_pad(sA, sTot[j - 1], len, q);
                lds_barrier();
                const int nj1 = A.w[j - 1];
                if (j == 1) nbm_mm(A.W[0], nj1, nj1, len, sList[0], nullptr, sA, sD, q);
                else nbm_mm(A.W[j - 1], nj1, sLen16[j - 2], len, sList[j - 1], sList[j - 2], sA, sD, q);
                if (q < nj1) {
                    // Lambda^(j-1) column q (0 for a stably inactive neuron: never used)
                    const int pc = j == 1 ? q : sPos[j - 2][q];
                    double* dst = lvb + A.lv_off[k][j - 1] + (size_t)r0 * nj1 + q;
                    for (int r = 0; r < nr; ++r) dst[(size_t)r * nj1] = pc >= 0 ? sD[pc * NBM_RS + r] : 0.0;
                }
            }
            if (k < L) {
                // concretise the rows: b_k + beta parts + Lambda^(0) c +/- |Lambda^(0)| rho
                if (q < n0) {
#pragma unroll
                    for (int r = 0; r < NBM_R; ++r) {
                        const double l0 = sD[q * NBM_RS + r];
                        bpart[r] += l0 * cq + sgn * fabs(l0) * rq;
                    }
                }
                const int wv = q >> 6;
#pragma unroll
                for (int r = 0; r < NBM_R; ++r) {
                    double x = bpart[r];
#pragma unroll
                    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
                    if ((q & 63) == 0) sA[wv * NBM_R + r] = x;
                }
                lds_barrier();
                if (q < nr) {
                    double x = A.b[k - 1][r0 + q];
                    for (int w2 = 0; w2 < NB_T / 64; ++w2) x += sA[w2 * NBM_R + q];
                    A.bd[ix_bd(box, k, upper ? 1 : 0) + r0 + q] = x;
                }
            }
            lds_barrier();
            continue;
        }
        // ---- reverse sweep of the block from the stored levels
        double y[NBM_R];
#pragma unroll
        for (int r = 0; r < NBM_R; ++r) {
            double yy = 0.0;
            if (r < nr) {
                if (k == L) yy = (upper ? A.g_hi : A.g_lo)[(A.u0 + box) * rows_k + sRow[r0 + r]];
                else yy = A.ub[ix_ub(box, k, upper ? 0 : 1) + sRow[r0 + r]];
            }
            y[r] = yy;
        }
        double jv[NBM_R];
#pragma unroll
        for (int r = 0; r < NBM_R; ++r) jv[r] = 0.0;
        if (k == L) {
            // rows of J = W_L D_{L-1} W_{L-1} ... D_1 W_1 (D = [z^ > 0]) for this block
            for (int j = L - 1; j >= 1; --j) {
                const int nj = A.w[j];
                if (q < nj) {
                    const double on = A.zn[ix_zn(box, j) + q] > 0.0 ? 1.0 : 0.0;
#pragma unroll
                    for (int r = 0; r < NBM_R; ++r) {
                        double x;
                        if (j == L - 1) x = r < nr ? Wk[(size_t)sRow[r0 + r] * nk1 + q] : 0.0;
                        else x = sD[q * NBM_RS + r];
                        sA[q * NBM_RS + r] = x * on;
                    }
                }
                lds_barrier();
                nbm_mm(A.W[j - 1], A.w[j - 1], A.w[j - 1], nj, nullptr, nullptr, sA, sD, q);
            }
            if (q < n0) {
#pragma unroll
                for (int r = 0; r < NBM_R; ++r) jv[r] = sD[q * NBM_RS + r];
            }
            lds_barrier();
        }
        if (q < n0) {
#pragma unroll
            for (int r = 0; r < NBM_R; ++r) {
                const double d = l0n[r] - jv[r];
                const double sd = d > 0.0 ? 1.0 : (d < 0.0 ? -1.0 : 0.0);
                cacc += y[r] * d;
                racc += sgn * y[r] * fabs(d);
                sA[q * NBM_RS + r] = y[r] * (cq + sgn * sd * rq);
            }
            // the next block's Lambda^(0) rows, in flight while this block runs
            const int r1 = r0 + NBM_R;
            const double* src = lvb + A.lv_off[k][0] + q;
#pragma unroll
            for (int r = 0; r < NBM_R; ++r) l0n[r] = r1 + r < rows ? src[(size_t)sRow[r1 + r] * n0] : 0.0;
        }
        lds_barrier();
        for (int j = 1; j <= k - 1; ++j) {
            const int nj = A.w[j];
            // this level's Lambda^(j) column, relaxation and bias, loaded before
            // the product so their latency overlaps it
            double lmv[NBM_R];
            double lo_j = 0.0, hi_j = 0.0, bj = 0.0;
            if (q < nj) {
                const double* src = j == k - 1 ? Wk + q : lvb + A.lv_off[k][j] + q;
                const size_t ld = j == k - 1 ? (size_t)nk1 : (size_t)nj;
#pragma unroll
                for (int r = 0; r < NBM_R; ++r) lmv[r] = r < nr ? src[(size_t)sRow[r0 + r] * ld] : 0.0;
                lo_j = A.bd[ix_bd(box, j, 0) + q];
                hi_j = A.bd[ix_bd(box, j, 1) + q];
                bj = A.b[j - 1][q];
            }
            // k over layer j-1: the inputs (all) or the listed neurons of a hidden layer
            // output columns over layer j's list
            if (j == 1) nbm_mm(A.WT[0], nj, sLen16[0], n0, nullptr, sList[0], sA, sD, q);
            else nbm_mm(A.WT[j - 1], nj, sLen16[j - 1], sLen[j - 2], sList[j - 2], sList[j - 1], sA, sD, q);
            const int pq = q < nj ? sPos[j - 1][q] : -1;
            if (j < k - 1) nbm_pad(sA, sTot[j - 1], sLen[j - 1], q);
            if (pq >= 0) {
                double s, t, a;
                nb_relax(lo_j, hi_j, s, t, a);
                double sa = 0.0, ta = 0.0;
#pragma unroll
                for (int r = 0; r < NBM_R; ++r) {
                    const double lm = lmv[r];
                    const bool sel = upper ? lm >= 0.0 : lm < 0.0;
                    const double obr = sD[pq * NBM_RS + r] + y[r] * bj;
                    if (sel) {
                        sa += obr * lm;
                        ta += y[r] * lm;
                    }
                    if (j < k - 1 && pq >= 0) sA[pq * NBM_RS + r] = obr * (sel ? s : a) + (sel ? y[r] * t : 0.0);
                }
                // j <= k - 1 <= L - 1 <= 3
                if (j == 1) { sacc[0] += sa; tacc[0] += ta; }
                else if (j == 2) { sacc[1] += sa; tacc[1] += ta; }
                else { sacc[2] += sa; tacc[2] += ta; }
            }
            lds_barrier();
        }
    }
    if (REV) {
        for (int j = 1; j <= k - 1; ++j) {
            if (q < A.w[j]) {
                const double sa = j == 1 ? sacc[0] : (j == 2 ? sacc[1] : sacc[2]);
                const double ta = j == 1 ? tacc[0] : (j == 2 ? tacc[1] : tacc[2]);
                A.st[ix_st(box, mode, j, 0) + q] += sa;
                A.st[ix_st(box, mode, j, 1) + q] += ta;
            }
        }
        if (q < n0) {
            A.cg[ix_cg(box, mode, 0) + q] += cacc;
            A.cg[ix_cg(box, mode, 1) + q] += racc;
        }
    }
}

// ---------------------------------------------------------------- reverse passes, 16 inputs
//
// The adjoint of one pass for networks with 16 inputs and at most three hidden layers,
// both directions of one box in a workgroup, 16 target rows at a time.  The products
// are formed transposed (A: weights of listed neurons, B: 16 rows), so that the
// accumulator of one level (lane l: neuron [4 i + l/16] of row [l%16]) becomes, after
// the relaxation's selection, the B operand of the next without leaving the registers:
//   level 1     Omega-bar_1 = W_1 Lambda-bar_0, four k-steps a tile;
//   last level  (j = k - 1) only enters through s-bar = sum_r sel Omega-bar Lambda, which is
//               linear in Omega-bar: each wave contracts the part of Omega-bar that its own
//               tiles of the level below contribute, and only the sums s-bar meet;
//   k = 3       a wave owns every fourth tile of level 1 and takes the last level's k-steps
//               of those tiles;
//   k = 4       every wave forms all of level 1 (a tenth of the pass), owns every fourth tile
//               of level 2 and takes the last level's k-steps of those.
// No barrier between the lists and the final sums.  Lists: the neurons that are not stably
// inactive of the levels below the last one, the unstable ones of the last (nothing is
// propagated past it, and s-bar and t-bar are used for those only), and the target rows
// with an adjoint (unstable neurons of a hidden target).
//
// What bounds it: the latency of the operand reads (the levels' rows from memory, the
// weights from L2) between short runs of MFMA (about 100 us of them at k = 3 and at
// k = 4), two waves a SIMD (k = 4: 256 registers, one spilled).  3,200 boxes of
// 16-256-256-256-12, k = 2, 3, 4: 69, 590,
// 385 us (one direction at a time through LDS with barriers at each level: 390, 1,126,
// 678; one direction a workgroup and three waves a SIMD: 99, 899, 568; the next rows and
// the next tile read ahead: 80, 590-680, 395).
constexpr int NR_PAD = NN_MAXW + 16;

struct RevLevel {                    // listed neurons of one level, zero past the end
    int idx[NR_PAD];
    double v[4][NR_PAD];             // s, t, a, bias (last level: bias only)
};

// Lists the kept neurons (one per lane, 256 lanes); returns their number.  Contains barriers.
__device__ __forceinline__ int rev_list(bool keep, int* idx, int* cnt, int& pos) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t bal = __ballot(keep);
    if (lane == 0) cnt[wave] = __popcll(bal);
    __syncthreads();
    int off = 0, n = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        off += q < wave ? cnt[q] : 0;
        n += cnt[q];
    }
    pos = keep ? off + __popcll(bal & ((1ull << lane) - 1ull)) : -1;
    if (keep) idx[pos] = tid;
    __syncthreads();                                     // cnt read
    return n;
}

template <int K>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) nn_rev_kernel(NbArgs A) {
    __shared__ RevLevel lev[K - 1];
    __shared__ int srow[NR_PAD], cnt[4];
    // s-bar, t-bar of levels with one owner a tile; the last level's s-bar one part a wave (k > 2)
    __shared__ double sst[K - 1][2][NR_PAD];
    __shared__ double spart[K > 2 ? 4 : 1][NR_PAD];
    const int box = blockIdx.x, tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (!A.ok[box]) return;
    const int L = A.L, M = A.w[K], wl = A.w[K - 1];
    const bool top = K == L;
    int pos, nrows, nlev[K - 1];
    {
        const double lo = !top && tid < M ? A.bd[ix_bd(box, K, 0) + tid] : 0.0;
        const double hi = !top && tid < M ? A.bd[ix_bd(box, K, 1) + tid] : 0.0;
        const int n = rev_list(tid < M && (top || (lo < 0.0 && hi > 0.0)), srow, cnt, pos);
        if (n == 0) return;                              // the same for every lane
        nrows = n;
    }
#pragma unroll
    for (int j = 1; j < K; ++j) {
        const int nj = A.w[j];
        const double lo = tid < nj ? A.bd[ix_bd(box, j, 0) + tid] : -1.0;
        const double hi = tid < nj ? A.bd[ix_bd(box, j, 1) + tid] : -1.0;
        RevLevel& v = lev[j - 1];
        const int n = rev_list(j == K - 1 ? lo < 0.0 && hi > 0.0 : lo >= 0.0 || hi > 0.0, v.idx, cnt, pos);
        if (pos >= 0) {
            double s, t, a;
            nb_relax(lo, hi, s, t, a);
            v.v[0][pos] = s; v.v[1][pos] = t; v.v[2][pos] = a; v.v[3][pos] = A.b[j - 1][tid];
        }
        if (tid < 16) {
            v.idx[n + tid] = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) v.v[q][n + tid] = 0.0;
        }
        for (int q = tid; q < NR_PAD; q += 256) {
            sst[j - 1][0][q] = sst[j - 1][1][q] = 0.0;
            if (j == K - 1) {
#pragma unroll
                for (int w = 0; w < (K > 2 ? 4 : 1); ++w) spart[w][q] = 0.0;
            }
        }
        nlev[j - 1] = n;
    }
    __syncthreads();
    const int nlast = nlev[K - 2], nut = (nlast + 15) >> 4, nt1 = (nlev[0] + 15) >> 4;
    const RevLevel& last = lev[K - 2];
    const double* WTk = A.WT[K - 1];                     // rows of W_k, transposed: [w_{k-1}][M]
    double* const lv = A.lv + (size_t)box * 2 * A.lv_bm;
    double cv[4], rv[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        cv[s] = A.cr[ix_cr(box, 0) + 4 * s + g];
        rv[s] = A.cr[ix_cr(box, 1) + 4 * s + g];
    }
    double cacc[4] = {0.0, 0.0, 0.0, 0.0}, racc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int r0 = 0; r0 < nrows; r0 += 16) {
        const int row = srow[r0 + r < nrows ? r0 + r : 0];
        // row seeds (0 past the last row), seeds of Lambda^(0), direct c and rho terms
        double y[2], seed[2][4];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            double v = top ? (m == 0 ? A.g_hi : A.g_lo)[(A.u0 + box) * M + row] : A.ub[ix_ub(box, K, m) + row];
            y[m] = r0 + r < nrows ? v : 0.0;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double jv = top ? A.jac[((size_t)box * M + row) * 16 + 4 * s + g] : 0.0;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const double sgn = m == 0 ? 1.0 : -1.0;
                const double d = lv[m * A.lv_bm + A.lv_off[K][0] + (size_t)row * 16 + 4 * s + g] - jv;
                const double sd = d > 0.0 ? 1.0 : (d < 0.0 ? -1.0 : 0.0);
                cacc[s] += y[m] * d;
                racc[s] += sgn * y[m] * fabs(d);
                seed[m][s] = y[m] * (cv[s] + sgn * sd * rv[s]);
            }
        }
        // Omega-bar of one tile of level 1 (listed neurons 16 t + 4 i + g)
        auto level1 = [&](const RevLevel& v, int t, nbd4 (&D)[2]) {
            const double* w = A.W[0] + (size_t)v.idx[16 * t + r] * 16 + g;
            double a[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) a[s] = w[4 * s];
            D[0] = D[1] = nbd4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int m = 0; m < 2; ++m) D[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], seed[m][s], D[m], 0, 0, 0);
        };
        // Lambda-bar of a tile of level j from its Omega-bar (in place), and, where `sums`, its
        // part of s-bar and t-bar
        auto select = [&](int j, const RevLevel& v, int t, nbd4 (&D)[2], bool sums) {
            const double* l0 = lv + A.lv_off[K][j] + (size_t)row * A.w[j];
            double lm[2][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = v.idx[16 * t + 4 * i + g];
#pragma unroll
                for (int m = 0; m < 2; ++m) lm[m][i] = l0[m * A.lv_bm + n];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = 16 * t + 4 * i + g;
                const double s = v.v[0][n], tt = v.v[1][n], a = v.v[2][n], b = v.v[3][n];
                double sa = 0.0, ta = 0.0;
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const bool sel = m == 0 ? lm[m][i] >= 0.0 : lm[m][i] < 0.0;
                    const double ob = D[m][i] + y[m] * b;
                    sa += sel ? ob * lm[m][i] : 0.0;
                    ta += sel ? y[m] * lm[m][i] : 0.0;
                    D[m][i] = ob * (sel ? s : a) + (sel ? y[m] * tt : 0.0);
                }
                if (sums) {
                    sa = sum16(sa);
                    ta = sum16(ta);
                    if (r == 0) {
                        sst[j - 1][0][n] += sa;
                        sst[j - 1][1][n] += ta;
                    }
                }
            }
        };
        // s-bar and t-bar of a tile of the last level from (this wave's part of) its Omega-bar;
        // whole: also the bias and t-bar terms
        auto finish = [&](int t, const nbd4 (&D)[2], bool whole, double* part) {
            double lm[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) lm[i] = WTk[(size_t)last.idx[16 * t + 4 * i + g] * M + row];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = 16 * t + 4 * i + g;
                const double yb = whole ? last.v[3][n] : 0.0;
                // upper pass selects lm >= 0, lower pass lm < 0
                const bool up = lm[i] >= 0.0;
                const double sa = sum16(((up ? D[0][i] : D[1][i]) + (up ? y[0] : y[1]) * yb) * lm[i]);
                if (whole) {
                    const double ta = sum16((up ? y[0] : y[1]) * lm[i]);
                    if (r == 0) sst[K - 2][1][n] += ta;
                }
                if (r == 0) part[n] += sa;
            }
        };
        if constexpr (K == 2) {
            for (int t = wave; t < nut; t += 4) {
                nbd4 D[2];
                level1(last, t, D);
                finish(t, D, true, sst[0][0]);
            }
        } else if constexpr (K == 3) {
            // own tiles of level 1, up to four tiles of the last level at a time (once even
            // if it has none, for the sums of level 1)
            const double* WT2 = A.WT[1];
            for (int t0 = 0; t0 == 0 || t0 < nut; t0 += 4) {
                nbd4 acc[4][2];
                int uc[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc[q][0] = acc[q][1] = nbd4{0.0, 0.0, 0.0, 0.0};
                    uc[q] = last.idx[t0 + q < nut ? 16 * (t0 + q) + r : 0];
                }
                for (int t = wave; t < nt1; t += 4) {
                    nbd4 D[2];
                    level1(lev[0], t, D);
                    double a[4][4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const double* w = WT2 + (size_t)lev[0].idx[16 * t + 4 * i + g] * wl;
#pragma unroll
                        for (int q = 0; q < 4; ++q) a[i][q] = w[uc[q]];
                    }
                    select(1, lev[0], t, D, t0 == 0);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (t0 + q >= nut) break;
#pragma unroll
                        for (int i = 0; i < 4; ++i)
#pragma unroll
                            for (int m = 0; m < 2; ++m)
                                acc[q][m] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][q], D[m][i], acc[q][m], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (t0 + q < nut) finish(t0 + q, acc[q], ((t0 + q) & 3) == wave, spart[wave]);
            }
        } else {
            // own tiles of level 2 over all of level 1
            const double* WT2 = A.WT[1];
            const double* WT3 = A.WT[2];
            const int w2 = A.w[2], nt2 = (nlev[1] + 15) >> 4, nmine = (nt2 - wave + 3) >> 2;
            nbd4 acc[4][2];
            int oc[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc[q][0] = acc[q][1] = nbd4{0.0, 0.0, 0.0, 0.0};
                oc[q] = lev[1].idx[q < nmine ? 16 * (wave + 4 * q) + r : 0];
            }
            for (int t = 0; t < nt1; ++t) {
                nbd4 D[2];
                level1(lev[0], t, D);
                double a[4][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const double* w = WT2 + (size_t)lev[0].idx[16 * t + 4 * i + g] * w2;
#pragma unroll
                    for (int q = 0; q < 4; ++q) a[i][q] = w[oc[q]];
                }
                select(1, lev[0], t, D, (t & 3) == wave);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (q >= nmine) break;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int m = 0; m < 2; ++m)
                            acc[q][m] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][q], D[m][i], acc[q][m], 0, 0, 0);
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q < nmine) select(2, lev[1], wave + 4 * q, acc[q], true);
            for (int t = 0; t < nut; ++t) {
                nbd4 D[2] = {nbd4{0.0, 0.0, 0.0, 0.0}, nbd4{0.0, 0.0, 0.0, 0.0}};
                const int u = last.idx[16 * t + r];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (q >= nmine) break;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const double a = WT3[(size_t)lev[1].idx[16 * (wave + 4 * q) + 4 * i + g] * wl + u];
#pragma unroll
                        for (int m = 0; m < 2; ++m)
                            D[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, acc[q][m][i], D[m], 0, 0, 0);
                    }
                }
                finish(t, D, (t & 3) == wave, spart[wave]);
            }
        }
    }
    __syncthreads();
    // the sums of both directions, into the upper direction's slots
#pragma unroll
    for (int j = 1; j < K; ++j) {
        if (tid >= nlev[j - 1]) continue;
        double s = sst[j - 1][0][tid];
        if (K > 2 && j == K - 1) {
#pragma unroll
            for (int w = 0; w < 4; ++w) s += spart[K > 2 ? w : 0][tid];
        }
        const int n = lev[j - 1].idx[tid];
        A.st[ix_st(box, 0, j, 0) + n] += s;
        A.st[ix_st(box, 0, j, 1) + n] += sst[j - 1][1][tid];
    }
    if (wave == 0) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double c = sum16(cacc[s]), h = sum16(racc[s]);
            if (r == 0) {
                A.cg[ix_cg(box, 0, 0) + 4 * s + g] += c;
                A.cg[ix_cg(box, 0, 1) + 4 * s + g] += h;
            }
        }
    }
}

// adjoints u-bar, l-bar of the bounds of hidden layer A.k from s-bar, t-bar
// (both pass directions, added in a fixed order)
__global__ void __launch_bounds__(NB_T) nb_radj_kernel(NbArgs A) {
    const int box = blockIdx.x, q = threadIdx.x, j = A.k;
    if (!A.ok[box] || q >= A.w[j]) return;
    const double sb = A.st[ix_st(box, 0, j, 0) + q] + A.st[ix_st(box, 1, j, 0) + q];
    const double tb = A.st[ix_st(box, 0, j, 1) + q] + A.st[ix_st(box, 1, j, 1) + q];
    const double lo = A.bd[ix_bd(box, j, 0) + q], hi = A.bd[ix_bd(box, j, 1) + q];
    double ubar = 0.0, lbar = 0.0;
    if (lo < 0.0 && hi > 0.0) {
        const double den = hi - lo, d2 = den * den;
        ubar = (-lo * sb + lo * lo * tb) / d2;
        lbar = (hi * sb - hi * hi * tb) / d2;
    }
    A.ub[ix_ub(box, j, 0) + q] = ubar;
    A.ub[ix_ub(box, j, 1) + q] = lbar;
}

// per box: c-bar, rho-bar (pass sums plus the layer-1 bounds, the neurons split over the
// lanes of an input and added in a fixed order), then the box and its clamps back to
// a~, sigma, mu.  3,200 boxes of 256 neurons: 23 us (one lane an input 140 us).
__global__ void __launch_bounds__(NB_T) nb_out_kernel(NbArgs A) {
    __shared__ double part[2][NB_T];
    const int box = blockIdx.x, tid = threadIdx.x;
    const int64_t unit = A.u0 + box;
    const int n0 = A.w[0], n1 = A.w[1];
    const int S = NB_T / n0, q = tid % n0, sl = tid / n0;
    const bool ok = A.ok[box] != 0u;
    double cb = 0.0, rb = 0.0;
    if (ok && sl < S) {
        const double* uu = A.ub + ix_ub(box, 1, 0);
        const double* ll = A.ub + ix_ub(box, 1, 1);
#pragma unroll 4
        for (int i = sl; i < n1; i += S) {
            const double w = A.W[0][(size_t)i * n0 + q];
            cb = __builtin_fma(w, uu[i] + ll[i], cb);
            rb = __builtin_fma(fabs(w), uu[i] - ll[i], rb);
        }
    }
    part[0][tid] = cb;
    part[1][tid] = rb;
    __syncthreads();
    if (tid >= n0) return;
    double ga = 0.0, gs = 0.0, gm = 0.0;
    if (ok) {
        cb = A.cg[ix_cg(box, 0, 0) + q] + A.cg[ix_cg(box, 1, 0) + q];
        rb = A.cg[ix_cg(box, 0, 1) + q] + A.cg[ix_cg(box, 1, 1) + q];
        for (int s = 0; s < S; ++s) {
            cb += part[0][s * n0 + q];
            rb += part[1][s * n0 + q];
        }
        const double sg = A.sigma[unit * n0 + q];
        const double mu = A.mu ? A.mu[unit * n0 + q] : 0.0;
        const double dlo_b = 0.5 * (cb - rb), dhi_b = 0.5 * (cb + rb);
        const bool lo_on = mu - sg < 0.0, hi_on = mu + sg > 0.0;
        ga = cb;
        gs = (lo_on ? -dlo_b : 0.0) + (hi_on ? dhi_b : 0.0);
        gm = (lo_on ? dlo_b : 0.0) + (hi_on ? dhi_b : 0.0);
    }
    if (q < A.nx) A.gz[unit * A.nx + q] = ga;
    else A.gv[unit * A.nu + (q - A.nx)] = ga;
    A.gsigma[unit * n0 + q] = gs;
    if (A.gmu) A.gmu[unit * n0 + q] = gm;
}

struct NbWorkspace {
    std::mutex mu;
    void* buf = nullptr;
    size_t cap = 0;
    WsFence fence;
};
static NbWorkspace g_nbws;

// VALU form: networks with four or more hidden layers (the MFMA form takes the rest)
template <bool REV>
static void nb_launch_pass(const NbArgs& a, int nb, hipStream_t st) {
    hipLaunchKernelGGL((nb_pass_kernel<REV, NN_MAXL - 1>), dim3((unsigned)nb, 2u), dim3(NB_T), 0, st, a);
}

extern "C" int leb_nn_backward(leb_mlp net, int32_t batch, int32_t N, const double* z, const double* v,
                               const double* mu, const double* sigma, const double* g_lo, const double* g_hi,
                               double* gz, double* gv, double* gmu, double* gsigma, void* stream) {
    if (!net) return LEB_EINVAL;
    if (batch < 0 || N < 0) return LEB_EINVAL;
    if (gmu && !mu) return LEB_EINVAL;
    const int64_t units = (int64_t)batch * N;
    if (units == 0) return LEB_OK;
    const int nx = net->nx, nu = net->nu;
    if (!sigma || !g_lo || !g_hi || !gsigma || (nx > 0 && (!z || !gz)) || (nu > 0 && (!v || !gv)))
        return LEB_EINVAL;
    const void* ptrs[] = {z, v, mu, sigma, g_lo, g_hi, gz, gv, gmu, gsigma};
    for (const void* p : ptrs)
        if (p && !aligned8(p)) return LEB_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    const int L = net->L;
    // stored levels of the passes: level j of pass k is w[k] x w[j]
    NbArgs a;
    memset(&a, 0, sizeof(a));
    // the MFMA form (at most three hidden layers) stores the output pass's levels too
    const bool use_mfma = L - 1 <= 3;
    size_t lv_bm = 0;
    for (int k = 2; k <= (use_mfma ? L : L - 1); ++k)
        for (int j = 0; j <= k - 2; ++j) {
            a.lv_off[k][j] = (int)lv_bm;
            lv_bm += (size_t)net->w[k] * net->w[j];
        }
    a.lv_bm = lv_bm;
    // per box: cr 2, zn L, bd 2L, st 4L, ub 2L, cg 4 rows of NN_MAXW doubles, the levels, the flag
    // (networks with 16 inputs: also the Jacobian's rows)
    const bool chain = use_mfma && net->w[0] == 16;
    const size_t jrows = chain ? (size_t)net->w[L] * net->w[0] : 0;
    const size_t per_box = (size_t)NN_MAXW * (2 + 9 * NN_MAXL + 4) + 2 * lv_bm + jrows;
    int64_t cb = (int64_t)(NB_LV_BUDGET / (per_box * sizeof(double)));
    cb = cb < NB_CHUNK_MIN ? NB_CHUNK_MIN : (cb > NB_CHUNK ? NB_CHUNK : cb);
    const int CB = (int)(units < cb ? units : cb);
    const size_t need = (size_t)CB * per_box * sizeof(double) + (size_t)CB * sizeof(uint32_t);
    std::lock_guard<std::mutex> lock(g_nbws.mu);
    if (need > g_nbws.cap) {
        if (g_nbws.buf) (void)hipFree(g_nbws.buf);
        g_nbws.buf = nullptr;
        g_nbws.cap = 0;
        if (getenv("LEB_TEST_FAIL_ALLOC") || hipMalloc(&g_nbws.buf, need) != hipSuccess) return LEB_ENOMEM;
        g_nbws.cap = need;
    }
    int rc;
    static DynLds lds;
    if ((rc = lds.raise((const void*)nb_box_group_kernel, NBG_LDS))) return rc;
    if ((rc = g_nbws.fence.enter(st))) return rc;
    WsFenceScope leave{g_nbws.fence, st};
    a.L = net->L;
    for (int l = 0; l <= net->L; ++l) a.w[l] = net->w[l];
    for (int l = 0; l < net->L; ++l) { a.W[l] = net->W[l]; a.WT[l] = net->WT[l]; a.b[l] = net->b[l]; }
    a.nx = nx; a.nu = nu;
    a.z = z; a.v = v; a.mu = mu; a.sigma = sigma; a.g_lo = g_lo; a.g_hi = g_hi;
    a.gz = gz; a.gv = gv; a.gmu = gmu; a.gsigma = gsigma;
    double* p = (double*)g_nbws.buf;
    a.cr = p; p += (size_t)CB * 2 * NN_MAXW;
    a.zn = p; p += (size_t)CB * NN_MAXL * NN_MAXW;
    a.bd = p; p += (size_t)CB * NN_MAXL * 2 * NN_MAXW;
    a.st = p; p += (size_t)CB * 2 * NN_MAXL * 2 * NN_MAXW;
    a.ub = p; p += (size_t)CB * NN_MAXL * 2 * NN_MAXW;
    a.cg = p; p += (size_t)CB * 2 * 2 * NN_MAXW;
    a.lv = p; p += (size_t)CB * 2 * lv_bm;
    a.jac = chain ? p : nullptr; p += (size_t)CB * jrows;
    a.ok = (uint32_t*)p;
    for (int64_t u0 = 0; u0 < units; u0 += CB) {
        const int nb = (int)((units - u0) < CB ? (units - u0) : CB);
        a.u0 = u0;
        if (nb >= NNG_MIN)
            hipLaunchKernelGGL(nb_box_group_kernel, dim3((unsigned)((nb + NNG_BOXES - 1) / NNG_BOXES)), dim3(NNG_T),
                               NBG_LDS, st, a, nb);
        else
            hipLaunchKernelGGL(nb_box_kernel, dim3((unsigned)nb), dim3(NB_T), 0, st, a);
        if (use_mfma) {
            const dim3 grid((unsigned)nb, 2u);
            for (int k = 2; k <= L; ++k) {
                a.k = k;
                if (chain && k < L) {
                    // one or two steps down to a 16-wide input: both directions together, levels of
                    // unstable rows only (3,200 boxes of 16-256-256-256-12: 1.65 ms for the
                    // two targets, 8.5 ms by the general pass); the rest below
                    HidArgs ha = {};
                    ha.WTt = net->WT[k - 1]; ha.bt = net->b[k - 1];
                    ha.W1 = net->W[0]; ha.b1 = net->b[0]; ha.W2 = net->W[1]; ha.b2 = net->b[1];
                    ha.w1 = net->w[1]; ha.w2 = net->w[2]; ha.M = net->w[k];
                    ha.lo = a.bd; ha.hi = a.bd + NN_MAXW;
                    ha.bstride = (size_t)NN_MAXL * 2 * NN_MAXW; ha.lstride = 2 * NN_MAXW;
                    ha.c = a.cr; ha.rho = a.cr + NN_MAXW; ha.cstride = 2 * NN_MAXW;
                    ha.lo_out = a.bd + (k - 1) * ha.lstride; ha.hi_out = ha.lo_out + NN_MAXW;
                    ha.lv = a.lv; ha.lv_bm = lv_bm; ha.off0 = a.lv_off[k][0]; ha.off1 = a.lv_off[k][1];
                    ha.ok = a.ok;
                    if (k == 2) hipLaunchKernelGGL(nn_hid1_kernel<true>, dim3(nb), dim3(256), 0, st, ha);
                    else hipLaunchKernelGGL(nn_hid2_kernel<true>, dim3((ha.M + 31) / 32, nb), dim3(256), 0, st, ha);
                    continue;
                }
                if (chain) {
                    // the output pass: both directions and the Jacobian's rows
                    ChainArgs ca = {};
                    ca.WTt = net->WT[L - 1]; ca.bt = net->b[L - 1];
                    for (int l = 0; l < L; ++l) { ca.W[l] = net->W[l]; ca.b[l] = net->b[l]; }
                    for (int l = 0; l <= L; ++l) ca.w[l] = net->w[l];
                    ca.k = L; ca.M = net->w[L]; ca.nbox = CB;
                    ca.lo = a.bd; ca.hi = a.bd + NN_MAXW;
                    ca.bstride = (size_t)NN_MAXL * 2 * NN_MAXW; ca.lstride = 2 * NN_MAXW;
                    ca.D = a.zn; ca.dbstride = (size_t)NN_MAXL * NN_MAXW; ca.dlstride = NN_MAXW;
                    ca.lv = a.lv; ca.lv_bm = lv_bm;
                    for (int l = 0; l + 2 <= L; ++l) ca.off[l] = a.lv_off[L][l];
                    ca.jac = a.jac; ca.jstride = jrows;
                    ca.ok = a.ok;
                    if ((rc = launch_nn_chain<true>(ca, 3, nb, st))) return rc;
                    continue;
                }
                hipLaunchKernelGGL(nbm_pass_kernel<false>, grid, dim3(NB_T), 0, st, a);
            }
            auto reverse = [&](int k) {
                a.k = k;
                if (!chain) hipLaunchKernelGGL(nbm_pass_kernel<true>, grid, dim3(NB_T), 0, st, a);
                else if (k == 2) hipLaunchKernelGGL(nn_rev_kernel<2>, dim3((unsigned)nb), dim3(NB_T), 0, st, a);
                else if (k == 3) hipLaunchKernelGGL(nn_rev_kernel<3>, dim3((unsigned)nb), dim3(NB_T), 0, st, a);
                else hipLaunchKernelGGL(nn_rev_kernel<4>, dim3((unsigned)nb), dim3(NB_T), 0, st, a);
            };
            reverse(L);
            for (int j = L - 1; j >= 1; --j) {
                a.k = j;
                hipLaunchKernelGGL(nb_radj_kernel, dim3((unsigned)nb), dim3(NB_T), 0, st, a);
                if (j >= 2) reverse(j);
            }
            hipLaunchKernelGGL(nb_out_kernel, dim3((unsigned)nb), dim3(NB_T), 0, st, a);
            continue;
        }
        for (int k = 2; k < L; ++k) {
            a.k = k;
            nb_launch_pass<false>(a, nb, st);
        }
        a.k = L;
        nb_launch_pass<true>(a, nb, st);
        for (int j = L - 1; j >= 1; --j) {
            a.k = j;
            hipLaunchKernelGGL(nb_radj_kernel, dim3((unsigned)nb), dim3(NB_T), 0, st, a);
            if (j >= 2) nb_launch_pass<true>(a, nb, st);
        }
        hipLaunchKernelGGL(nb_out_kernel, dim3((unsigned)nb), dim3(NB_T), 0, st, a);
    }
    return hipGetLastError() == hipSuccess ? LEB_OK : LEB_EDEVICE;
}

}  // namespace leb
