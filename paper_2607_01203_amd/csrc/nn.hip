// nn.hip -- linearization-error bound for ReLU-MLP dynamics (section IV.B).
//
// Dynamics f(x, u) = x + g([x; u]) (or g alone), g a ReLU MLP
//   z_l = W_l a_{l-1} + b_l, a_l = relu(z_l), g = z_L.
// CROWN (Theorem "CROWN bounds", Zhang et al. Thm 3.2) gives affine bounds
// W_lo a + b_lo <= g(a) <= W_hi a + b_hi over the box; Theorem 2 turns them
// into the remainder bound with the local Jacobian J = J_g(a~):
//   r_hi = max_X (W_hi - J) a + J a~ - g(a~) + b_hi, r_lo = min_X (...lo...).
// Relaxations per neuron from pre-activation bounds [l, u]: active (l >= 0)
// identity, inactive (u <= 0) zero, unstable: upper line s z + t with
// s = u/(u-l), t = -s l, lower line a z with a = 1 iff u >= -l.  First-layer
// bounds are exact; every later hidden layer gets its own full CROWN pass.
//
// GPU design.  Each backward substitution step
//     Lambda_next = (Lambda (.) S) W_l      (S sign-selected slopes)
// is a batched dense contraction run on FP64 MFMA (v_mfma_f64_16x16x4): the
// operand is generated on the fly from Lambda and the per-box slopes, the weights
// come from L2, and the per-row bias (intercepts, Omega b_l) and rounding-term
// weights are accumulated beside.  Kernels (nn_hid.hpp, shared with the adjoint): hidden
// targets of 16-input networks run both directions together; every other chain
// runs one mode (upper, lower, Jacobian with S = 1[z^ > 0]) a workgroup.
//
// Soundness in floating point: every FP64 dot product of length <= 300 has
// error <= 2^-44.8 times the dot product of absolute values.  Each bound
// adds 2^-40 times the absolute-value dot products of every step (computed
// alongside as matrix-vector products), covering the relaxation scaling,
// the contraction, the bias sums, the concretisation, the nominal forward
// pass and the Jacobian chain.  Upper-line slopes are rounded up so the
// computed line stays above the ReLU on [l, u].
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <mutex>
#include <vector>

#include "leb.h"
#include "leb_internal.hpp"

#include "nn_net.hpp"
#include "nn_hid.hpp"

namespace leb {

constexpr int NN_CHUNK = 4096;   // boxes per pass
constexpr uint32_t NN_UNSTABLE = 1u << 31;   // private per-box bit: some neuron is unstable

}  // namespace leb

namespace leb {

// ------------------------------------------------------------------ prep

struct PrepArgs {
    const double* z; const double* v; const double* mu; const double* sigma;
    int64_t u0; int nbox, nact;                            // boxes of the chunk's buffers, of this launch
    int L; int w[NN_MAXL + 1]; int nx, nu;
    const double* W[NN_MAXL]; const double* WT[NN_MAXL]; const double* b[NN_MAXL];
    // outputs (chunk-local)
    double* alpha; double* c; double* rho;                 // [box][w0]
    double* zhat;                                          // [L-1][box][W]
    double* lo; double* hi;                                // [L-1][box][W] (layer 1 filled here)
    double* s; double* t; double* a; double* D; double* e; double* amax;   // layer 1's relaxation, [box][W]
    double* g; double* eg;                                 // [box][m]
    uint32_t* flags;                                       // [box]
};

// Relaxation coefficients of one neuron with bounds [l, u] (s rounded up: the line stays above
// relu on [l, u])
__device__ __forceinline__ void relax_coeffs(double l, double u, double& s, double& t, double& a) {
    if (l >= 0.0) { s = 1.0; t = 0.0; a = 1.0; }
    else if (u <= 0.0) { s = 0.0; t = 0.0; a = 0.0; }
    else {
        s = u / (u - l);
        s = s + s * 0x1p-50;
        t = -s * l;
        t = t + t * 0x1p-50;
        a = (u >= -l) ? 1.0 : 0.0;
    }
}

// Layer 1's relaxation of one neuron at offset o: bounds [l, u], wa = |W_1| (|c| + rho) + |b|
// (the sums of its bounds; the layers above take nn_relax_kernel)
__device__ __forceinline__ void relax1_store(const PrepArgs& A, size_t o, double l, double u, double wa) {
    double s, t, a;
    relax_coeffs(l, u, s, t, a);
    A.lo[o] = l; A.hi[o] = u;
    A.s[o] = s; A.t[o] = t; A.a[o] = a;
    A.e[o] = fmax(fabs(l), fabs(u)) + wa + fabs(t);
    A.amax[o] = fmax(u, 0.0);
}

// one workgroup (256 lanes) per box
__global__ void __launch_bounds__(256) nn_prep_kernel(PrepArgs A) {
    __shared__ double s_a[NN_MAXW], s_m[NN_MAXW], s_v[NN_MAXW];
    __shared__ double s_c[NN_MAXW], s_r[NN_MAXW], s_al[NN_MAXW];
    __shared__ uint32_t s_flag, s_uns;
    const int box = blockIdx.x, q = threadIdx.x;
    const int64_t unit = A.u0 + box;
    const int n0 = A.w[0], m = A.w[A.L];
    if (q == 0) s_flag = s_uns = 0;
    __syncthreads();
    if (q < n0) {
        const double x = q < A.nx ? A.z[unit * A.nx + q] : A.v[unit * A.nu + (q - A.nx)];
        const double sg = A.sigma[unit * n0 + q];
        const double mu = A.mu ? A.mu[unit * n0 + q] : 0.0;
        uint32_t f = 0;
        if (!isfinite(x) || !isfinite(sg) || !isfinite(mu) || !(sg >= 0.0)) f |= LEB_FLAG_BAD_INPUT;
        if (fabs(mu) > sg) f |= LEB_FLAG_HULL_EXTENDED;
        if (f) atomicOr(&s_flag, f);
        // box = hull({a~}, a~ + mu +/- sigma): centre and half-width, widened
        // so the FP64 box encloses the exact one
        const double dlo = fmin(mu - sg, 0.0), dhi = fmax(mu + sg, 0.0);
        const double cc = x + 0.5 * (dlo + dhi);
        double rr = 0.5 * (dhi - dlo);
        rr = rr + rr * 0x1p-50 + (fabs(x) + fabs(dlo) + fabs(dhi)) * 0x1p-51;
        s_al[q] = x; s_c[q] = cc; s_r[q] = rr;
        s_a[q] = x;                                   // forward input
        s_m[q] = fabs(x);                             // magnitude chain (nominal pass error)
        s_v[q] = fabs(cc - x) + rr;                   // |a - a~| bound (Jacobian error)
        A.alpha[box * n0 + q] = x; A.c[box * n0 + q] = cc; A.rho[box * n0 + q] = rr;
    }
    __syncthreads();
    // first layer bounds, exact affine image of the box
    {
        const int h = A.w[1];
        if (q < h) {
            const double* Wr = A.W[0] + (size_t)q * n0;
            double lin = A.b[0][q], mag = 0.0, abs_ = fabs(A.b[0][q]);
            for (int k = 0; k < n0; ++k) {
                lin = __builtin_fma(Wr[k], s_c[k], lin);
                mag = __builtin_fma(fabs(Wr[k]), s_r[k], mag);
                abs_ = __builtin_fma(fabs(Wr[k]), fabs(s_c[k]), abs_);
            }
            const double err = RT * (abs_ + mag + fabs(lin));
            const double l = lin - mag - err, u = lin + mag + err;
            relax1_store(A, (size_t)box * NN_MAXW + q, l, u, abs_ + mag);
            if (l < 0.0 && u > 0.0) s_uns = 1u;
        }
    }
    // nominal forward pass, magnitude chains (nominal error, Jacobian error)
    for (int l = 0; l < A.L; ++l) {
        const int in = A.w[l], out = A.w[l + 1];
        double z = 0.0, mz = 0.0, vz = 0.0;
        if (q < out) {
            const double* WT = A.WT[l];
            z = A.b[l][q];
            mz = fabs(A.b[l][q]);
            // eight k at a time, the weight loads of a group issued before its sums
            int k = 0;
            for (; k + 8 <= in; k += 8) {
                double wv[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) wv[u] = WT[(size_t)(k + u) * out + q];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    z = __builtin_fma(wv[u], s_a[k + u], z);
                    mz = __builtin_fma(fabs(wv[u]), s_m[k + u], mz);
                    vz = __builtin_fma(fabs(wv[u]), s_v[k + u], vz);
                }
            }
            for (; k < in; ++k) {
                const double wk = WT[(size_t)k * out + q];
                z = __builtin_fma(wk, s_a[k], z);
                mz = __builtin_fma(fabs(wk), s_m[k], mz);
                vz = __builtin_fma(fabs(wk), s_v[k], vz);
            }
        }
        __syncthreads();
        if (q < out) {
            if (l < A.L - 1) {
                const bool on = z > 0.0;
                A.zhat[((size_t)l * A.nbox + box) * NN_MAXW + q] = z;
                if (l == 0) A.D[(size_t)box * NN_MAXW + q] = on ? 1.0 : 0.0;
                s_a[q] = on ? z : 0.0;
                s_m[q] = mz;
                s_v[q] = on ? vz : 0.0;
            } else {
                A.g[box * m + q] = z;
                // |g^ - g| and |(J^ - J)(a - a~)| allowances
                A.eg[box * m + q] = RT * (mz + vz);
            }
        }
        __syncthreads();
    }
    if (q == 0) A.flags[box] = s_flag | (s_uns ? NN_UNSTABLE : 0u);
}

// ---------------------------------------------------------------- relax

struct RelaxArgs {
    const double* lo; const double* hi;     // [box][W] of layer l
    const double* amax_prev;                // [box][W] of layer l-1
    const double* WT;                       // layer l transposed [w[l-1]][w[l]]
    const double* b;                        // [w[l]]
    const double* zhat;                     // [box][W]
    int in, out, nact;
    double* s; double* t; double* a; double* D; double* e; double* amax;   // [box][W]
    uint32_t* boxflags;                     // [box]
};

// sound relaxation coefficients and rounding weights e = zmax + |W| amax_prev + |b| + |t|
__global__ void __launch_bounds__(256) nn_relax_kernel(RelaxArgs A) {
    __shared__ double s_am[NN_MAXW];
    const int box = blockIdx.x, q = threadIdx.x;
    if (q < A.in) {
        s_am[q] = A.amax_prev[(size_t)box * NN_MAXW + q];
    }
    __syncthreads();
    const size_t o = (size_t)box * NN_MAXW + q;
    const bool unstable = q < A.out && A.lo[o] < 0.0 && A.hi[o] > 0.0;
    if (__syncthreads_or(unstable) && q == 0) atomicOr(&A.boxflags[box], NN_UNSTABLE);
    if (q >= A.out) return;
    const double l = A.lo[o], u = A.hi[o];
    double s, t, a;
    relax_coeffs(l, u, s, t, a);
    double wa = 0.0;
    int k = 0;
    for (; k + 8 <= A.in; k += 8) {           // the weight loads of a group issued before its sums
        double wv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) wv[u] = A.WT[(size_t)(k + u) * A.out + q];
#pragma unroll
        for (int u = 0; u < 8; ++u) wa = __builtin_fma(fabs(wv[u]), s_am[k + u], wa);
    }
    for (; k < A.in; ++k) wa = __builtin_fma(fabs(A.WT[(size_t)k * A.out + q]), s_am[k], wa);
    A.s[o] = s; A.t[o] = t; A.a[o] = a;
    A.D[o] = A.zhat[o] > 0.0 ? 1.0 : 0.0;
    A.e[o] = fmax(fabs(l), fabs(u)) + wa + fabs(A.b[q]) + fabs(t);
    A.amax[o] = fmax(u, 0.0);
}

// ---------------------------------------------------------- 16 boxes a workgroup
//
// nn_prep_kernel and nn_relax_kernel read every weight of the network for one box; with
// many boxes that is what they wait for (3,200 boxes of 16-256-256-256-12: 3.4 GB from
// L2 for each).  The forms below take 16 boxes as the columns of FP64 MFMA
// (v_mfma_f64_16x16x4: Y^T = W X^T, A: a weight tile from W^T, B: 16 boxes' inputs in
// LDS).  The instruction adds its four products in order, each rounded, so every sum
// is bitwise the fused-multiply-add chain of the one-box kernels.
//
// Eight waves, wave w the output tiles w and w + 8.  What bounds them: MFMA at one
// workgroup a compute unit (three chains of 256 x 256 products, 41 us for prep at 200
// workgroups).  3,200 boxes: prep 93 us (one box a workgroup: 250; four boxes on the
// VALU, bound by broadcast reads of LDS: 197), relax 27 us (102; 47).  The whole bound with
// the grouped and the one-box form: 235 and 144 us at 50 boxes, 452 and 391 at 400, 692
// and 693 at 800, 1,138 and 1,228 at 1,600, 2,048 and 2,343 at 3,200.
constexpr size_t NNG_LDS = (size_t)3 * NN_MAXW * NNG_RS * sizeof(double);

__global__ void __launch_bounds__(NNG_T) nn_prep_group_kernel(PrepArgs A) {
    extern __shared__ __attribute__((aligned(16))) double X[];       // [3][NN_MAXW][NNG_RS]
    __shared__ uint32_t s_flag[NNG_BOXES], s_uns[NNG_BOXES];
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = blockIdx.x * NNG_BOXES, nb = min(NNG_BOXES, A.nact - b0);
    const int n0 = A.w[0], m = A.w[A.L];
    auto X_ = [&](int c, int n, int b) -> double& { return X[(c * NN_MAXW + n) * NNG_RS + b]; };
    if (tid < NNG_BOXES) s_flag[tid] = s_uns[tid] = 0;
    __syncthreads();
    // box = hull({a~}, a~ + mu +/- sigma): centre and half-width, widened so the FP64 box
    // encloses the exact one; planes: centre, its magnitude, half-width
    for (int e = tid; e < NNG_BOXES * n0; e += NNG_T) {
        const int b = e / n0, q = e - b * n0, box = b0 + min(b, nb - 1);
        const int64_t unit = A.u0 + box;
        const double x = q < A.nx ? A.z[unit * A.nx + q] : A.v[unit * A.nu + (q - A.nx)];
        const double sg = A.sigma[unit * n0 + q];
        const double mu = A.mu ? A.mu[unit * n0 + q] : 0.0;
        uint32_t f = 0;
        if (!isfinite(x) || !isfinite(sg) || !isfinite(mu) || !(sg >= 0.0)) f |= LEB_FLAG_BAD_INPUT;
        if (fabs(mu) > sg) f |= LEB_FLAG_HULL_EXTENDED;
        if (f) atomicOr(&s_flag[b], f);
        const double dlo = fmin(mu - sg, 0.0), dhi = fmax(mu + sg, 0.0);
        const double cc = x + 0.5 * (dlo + dhi);
        double rr = 0.5 * (dhi - dlo);
        rr = rr + rr * 0x1p-50 + (fabs(x) + fabs(dlo) + fabs(dhi)) * 0x1p-51;
        X_(0, q, b) = cc; X_(1, q, b) = fabs(cc); X_(2, q, b) = rr;
        if (b < nb) { A.alpha[box * n0 + q] = x; A.c[box * n0 + q] = cc; A.rho[box * n0 + q] = rr; }
    }
    __syncthreads();
    // l = -1: first layer bounds, exact affine image of the box (planes lin, abs, mag);
    // l >= 0: nominal forward pass, magnitude chains (nominal error, Jacobian error)
    for (int l = -1; l < A.L; ++l) {
        const int in = A.w[l < 0 ? 0 : l], out = A.w[l < 0 ? 1 : l + 1];
        const double* W = A.WT[l < 0 ? 0 : l];
        const double* bias = A.b[l < 0 ? 0 : l];
        const bool last = l == A.L - 1;
        d4 acc[2][3];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = 16 * (wave + 8 * q) + 4 * i + g;
                const double b = n < out ? bias[n] : 0.0;
                acc[q][0][i] = b;
                acc[q][1][i] = fabs(b);
                acc[q][2][i] = 0.0;
            }
        if (l <= 0) group_products<3, true, false>(W, in, out, X, wave, r, g, acc);
        else group_products<3, true, true>(W, in, out, X, wave, r, g, acc);
        __syncthreads();                                     // the inputs are read
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (16 * (wave + 8 * q) >= out) break;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = 16 * (wave + 8 * q) + 4 * i + g;
                const double z = acc[q][0][i], mz = acc[q][1][i], vz = acc[q][2][i];
                if (l < 0) {
                    const double err = RT * (mz + vz + fabs(z));
                    X_(0, n, r) = z - vz - err;
                    X_(1, n, r) = z + vz + err;
                    X_(2, n, r) = mz + vz;
                } else if (!last) {
                    X_(0, n, r) = z;
                    X_(1, n, r) = mz;
                    X_(2, n, r) = vz;
                } else if (r < nb && n < out) {
                    A.g[(b0 + r) * m + n] = z;
                    // |g^ - g| and |(J^ - J)(a - a~)| allowances
                    A.eg[(b0 + r) * m + n] = RT * (mz + vz);
                }
            }
        }
        __syncthreads();
        if (l < 0) {
            for (int e = tid; e < nb * out; e += NNG_T) {
                const int b = e / out, n = e - b * out;
                const double lo = X_(0, n, b), hi = X_(1, n, b);
                relax1_store(A, (size_t)(b0 + b) * NN_MAXW + n, lo, hi, X_(2, n, b));
                if (lo < 0.0 && hi > 0.0) s_uns[b] = 1u;
            }
            __syncthreads();
            // planes of the forward pass: input, its magnitude, |a - a~| bound
            for (int e = tid; e < NNG_BOXES * n0; e += NNG_T) {
                const int b = e / n0, q = e - b * n0, box = b0 + min(b, nb - 1);
                const double x = A.alpha[box * n0 + q];
                X_(0, q, b) = x; X_(1, q, b) = fabs(x);
                X_(2, q, b) = fabs(A.c[box * n0 + q] - x) + A.rho[box * n0 + q];
            }
            __syncthreads();
        } else if (!last) {
            for (int e = tid; e < nb * out; e += NNG_T) {
                const int b = e / out, n = e - b * out;
                const double z = X_(0, n, b);
                A.zhat[((size_t)l * A.nbox + b0 + b) * NN_MAXW + n] = z;
                if (l == 0) A.D[(size_t)(b0 + b) * NN_MAXW + n] = z > 0.0 ? 1.0 : 0.0;
            }
        }
    }
    if (tid < nb) A.flags[b0 + tid] = s_flag[tid] | (s_uns[tid] ? NN_UNSTABLE : 0u);
}

__global__ void __launch_bounds__(NNG_T) nn_relax_group_kernel(RelaxArgs A) {
    __shared__ double X[NN_MAXW * NNG_RS];
    __shared__ uint32_t s_uns[NNG_BOXES];
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = blockIdx.x * NNG_BOXES, nb = min(NNG_BOXES, A.nact - b0);
    if (tid < NNG_BOXES) s_uns[tid] = 0;
    for (int e = tid; e < NNG_BOXES * A.in; e += NNG_T) {
        const int b = e / A.in, q = e - b * A.in, box = b0 + min(b, nb - 1);
        X[q * NNG_RS + b] = A.amax_prev[(size_t)box * NN_MAXW + q];
    }
    __syncthreads();
    d4 acc[2][1];
    acc[0][0] = acc[1][0] = d4{0.0, 0.0, 0.0, 0.0};
    group_products<1, false, false>(A.WT, A.in, A.out, X, wave, r, g, acc);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (16 * (wave + 8 * q) >= A.out) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) X[(16 * (wave + 8 * q) + 4 * i + g) * NNG_RS + r] = acc[q][0][i];
    }
    __syncthreads();
    for (int e = tid; e < nb * A.out; e += NNG_T) {
        const int b = e / A.out, q = e - b * A.out;
        const size_t o = (size_t)(b0 + b) * NN_MAXW + q;
        const double l = A.lo[o], u = A.hi[o];
        if (l < 0.0 && u > 0.0) s_uns[b] = 1u;
        double s, t, a;
        relax_coeffs(l, u, s, t, a);
        A.s[o] = s; A.t[o] = t; A.a[o] = a;
        A.D[o] = A.zhat[o] > 0.0 ? 1.0 : 0.0;
        A.e[o] = fmax(fabs(l), fabs(u)) + X[q * NNG_RS + b] + fabs(A.b[q]) + fabs(t);
        A.amax[o] = fmax(u, 0.0);
    }
    __syncthreads();
    if (tid < nb && s_uns[tid]) A.boxflags[b0 + tid] |= NN_UNSTABLE;
}

// ----------------------------------------------------------- concretize

struct ConcArgs {
    const double* L0;            // [mode][box][M][n0]
    const double* beta; const double* eps;   // [mode][box][M]
    const double* c; const double* rho;      // [box][n0]
    int M, n0, nbox;
    double* lo; double* hi;      // [box][W]
};

// mode 0 -> upper bound into hi, mode 1 -> lower bound into lo
__global__ void __launch_bounds__(256) nn_concretize_kernel(ConcArgs A) {
    const int box = blockIdx.x, r = threadIdx.x, mode = blockIdx.y;
    if (r >= A.M) return;
    const double* Lr = A.L0 + (((size_t)mode * A.nbox + box) * A.M + r) * A.n0;
    const double* c = A.c + (size_t)box * A.n0;
    const double* rho = A.rho + (size_t)box * A.n0;
    double lin = 0.0, mag = 0.0, ab = 0.0;
    // eight k at a time, every load of a group issued before its sums (same order of summation)
    int k = 0;
    for (; k + 8 <= A.n0; k += 8) {
        double lv[8], cv[8], rv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) { lv[u] = Lr[k + u]; cv[u] = c[k + u]; rv[u] = rho[k + u]; }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            lin = __builtin_fma(lv[u], cv[u], lin);
            mag = __builtin_fma(fabs(lv[u]), rv[u], mag);
            ab = __builtin_fma(fabs(lv[u]), fabs(cv[u]), ab);
        }
    }
    for (; k < A.n0; ++k) {
        lin = __builtin_fma(Lr[k], c[k], lin);
        mag = __builtin_fma(fabs(Lr[k]), rho[k], mag);
        ab = __builtin_fma(fabs(Lr[k]), fabs(c[k]), ab);
    }
    const size_t o = ((size_t)mode * A.nbox + box) * A.M + r;
    const double beta = A.beta[o];
    const double err = RT * (A.eps[o] + ab + mag + fabs(beta) + fabs(lin));
    if (mode == 0) A.hi[(size_t)box * NN_MAXW + r] = lin + mag + beta + err;
    else A.lo[(size_t)box * NN_MAXW + r] = lin - mag + beta - err;
}

// ---------------------------------------------------------------- thm 2

struct Thm2Args {
    const double* L0;            // [3][box][m][n0]: upper, lower, Jacobian
    const double* beta; const double* eps;   // [3][box][m]
    const double* alpha; const double* c; const double* rho;   // [box][n0]
    const double* g; const double* eg;        // [box][m]
    const uint32_t* flags;       // [box]
    const double* Juser;         // NULL, or the caller's J [unit][m][n0] (replaces mode 2)
    int m, n0, nbox;
    int64_t u0;
    double* r_lo; double* r_hi; double* c_bar; double* rho_bar; double pad;
    uint32_t* flags_out;
};

__global__ void __launch_bounds__(64) nn_thm2_kernel(Thm2Args A) {
    const int box = blockIdx.x, i = threadIdx.x;
    if (i >= A.m) return;
    const size_t sz = (size_t)A.nbox * A.m;
    const double* Lu = A.L0 + ((size_t)0 * sz + (size_t)box * A.m + i) * A.n0;
    const double* Ll = A.L0 + ((size_t)1 * sz + (size_t)box * A.m + i) * A.n0;
    const double* J = A.Juser ? A.Juser + ((size_t)(A.u0 + box) * A.m + i) * A.n0
                              : A.L0 + ((size_t)2 * sz + (size_t)box * A.m + i) * A.n0;
    const double* al = A.alpha + (size_t)box * A.n0;
    const double* c = A.c + (size_t)box * A.n0;
    const double* rho = A.rho + (size_t)box * A.n0;
    double hu = 0.0, hl = 0.0, mu_ = 0.0, ml = 0.0, ja = 0.0, ab = 0.0;
    for (int k = 0; k < A.n0; ++k) {
        const double du = Lu[k] - J[k], dl = Ll[k] - J[k];
        hu = __builtin_fma(du, c[k], hu);
        hl = __builtin_fma(dl, c[k], hl);
        mu_ = __builtin_fma(fabs(du), rho[k], mu_);
        ml = __builtin_fma(fabs(dl), rho[k], ml);
        ja = __builtin_fma(J[k], al[k], ja);
        ab += (fabs(du) + fabs(dl)) * fabs(c[k]) + fabs(J[k]) * fabs(al[k]);
    }
    const size_t ou = (size_t)box * A.m + i, ol = sz + ou;
    const double g = A.g[ou];
    const double bu = A.beta[ou], bl = A.beta[ol];
    const double base = ja - g;
    double hi = hu + mu_ + base + bu;
    double lo = hl - ml + base + bl;
    const double common = ab + mu_ + ml + fabs(ja) + fabs(g);
    hi += RT * (A.eps[ou] + common + fabs(bu) + fabs(hi)) + A.eg[ou];
    lo -= RT * (A.eps[ol] + common + fabs(bl) + fabs(lo)) + A.eg[ou];
    // 0 = r(a~) lies in every valid bound (for any J)
    hi = fmax(hi, 0.0);
    lo = fmin(lo, 0.0);
    uint32_t f = A.flags[box];
    // no unstable neuron: g is affine on the box and equal to its linearization
    // with the computed Jacobian, so that remainder is exactly 0
    if (!(f & NN_UNSTABLE) && !A.Juser) { lo = 0.0; hi = 0.0; }
    // a caller's J with a non-finite entry in this row: the whole unit is invalid
    if (A.Juser) {
        const double* Jb = A.Juser + (size_t)(A.u0 + box) * A.m * A.n0;
        bool bad = false;
        for (int q = 0; q < A.m * A.n0; ++q) bad |= !isfinite(Jb[q]);
        if (bad) f |= LEB_FLAG_BAD_INPUT;
    }
    if (f & LEB_FLAG_BAD_INPUT) { lo = -INFINITY; hi = INFINITY; }
    const int64_t o = (A.u0 + box) * A.m + i;
    A.r_lo[o] = lo;
    A.r_hi[o] = hi;
    if (A.c_bar) {
        double cb, rb;
        if (isfinite(lo) && isfinite(hi)) {
            cb = 0.5 * (lo + hi);
            rb = fmax(hi - cb, cb - lo);
            rb = rb + fabs(rb) * 0x1p-50 + A.pad;
        } else { cb = 0.0; rb = INFINITY; }
        A.c_bar[o] = cb;
        A.rho_bar[o] = rb;
    }
    if (A.flags_out && i == 0) A.flags_out[A.u0 + box] = f & ~NN_UNSTABLE;
}

// --------------------------------------------------------------- host

struct NNWorkspace {
    std::mutex mu;
    std::vector<void*> bufs;
    std::vector<size_t> sizes;
    WsFence fence;
};
static NNWorkspace g_nnws;

static int nn_ws(int slot, size_t bytes, double** out) {
    if ((int)g_nnws.bufs.size() <= slot) { g_nnws.bufs.resize(slot + 1, nullptr); g_nnws.sizes.resize(slot + 1, 0); }
    if (g_nnws.sizes[slot] < bytes) {
        if (g_nnws.bufs[slot]) (void)hipFree(g_nnws.bufs[slot]);
        g_nnws.bufs[slot] = nullptr;
        g_nnws.sizes[slot] = 0;
        if (getenv("LEB_TEST_FAIL_ALLOC")) return LEB_ENOMEM;
        if (hipMalloc(&g_nnws.bufs[slot], bytes) != hipSuccess) return LEB_ENOMEM;
        g_nnws.sizes[slot] = bytes;
    }
    *out = (double*)g_nnws.bufs[slot];
    return LEB_OK;
}

}  // namespace leb

using namespace leb;

extern "C" int leb_mlp_create(int32_t n_layers, const int32_t* widths, const float* const* W,
                              const float* const* b, int32_t nx, int32_t residual, leb_mlp* out) {
    if (!out || !widths || !W || !b) return LEB_EINVAL;
    *out = nullptr;
    if (n_layers < 2 || n_layers > NN_MAXL) return LEB_ENOTSUP;
    for (int l = 0; l <= n_layers; ++l)
        if (widths[l] < 1) return LEB_EINVAL;
    for (int l = 0; l < n_layers; ++l) {
        if (widths[l] > NN_MAXW || widths[l] % 16 != 0) return LEB_ENOTSUP;
        if (!W[l] || !b[l]) return LEB_EINVAL;
    }
    if (widths[n_layers] > 64) return LEB_ENOTSUP;
    if (nx < 0 || nx > widths[0]) return LEB_EINVAL;
    if (residual && nx != widths[n_layers]) return LEB_EINVAL;
    leb_mlp_s* net = new leb_mlp_s();
    net->L = n_layers;
    for (int l = 0; l <= n_layers; ++l) net->w[l] = widths[l];
    net->nx = nx;
    net->nu = widths[0] - nx;
    net->residual = residual ? 1 : 0;
    for (int l = 0; l < n_layers; ++l) {
        const int in = widths[l], o = widths[l + 1];
        std::vector<double> w((size_t)in * o), wt((size_t)in * o), bb(o);
        for (int r = 0; r < o; ++r) {
            for (int k = 0; k < in; ++k) {
                const double x = (double)W[l][(size_t)r * in + k];
                if (!isfinite(x)) { leb_mlp_destroy(net); return LEB_EINVAL; }
                w[(size_t)r * in + k] = x;
                wt[(size_t)k * o + r] = x;
            }
            bb[r] = (double)b[l][r];
            if (!isfinite(bb[r])) { leb_mlp_destroy(net); return LEB_EINVAL; }
        }
        void *p1 = nullptr, *p2 = nullptr, *p3 = nullptr;
        if (getenv("LEB_TEST_FAIL_ALLOC") || hipMalloc(&p1, w.size() * 8) != hipSuccess ||
            hipMalloc(&p2, wt.size() * 8) != hipSuccess || hipMalloc(&p3, bb.size() * 8) != hipSuccess) {
            if (p1) (void)hipFree(p1);
            if (p2) (void)hipFree(p2);
            if (p3) (void)hipFree(p3);
            leb_mlp_destroy(net);
            return LEB_ENOMEM;
        }
        net->allocs.push_back(p1); net->allocs.push_back(p2); net->allocs.push_back(p3);
        if (hipMemcpy(p1, w.data(), w.size() * 8, hipMemcpyHostToDevice) != hipSuccess ||
            hipMemcpy(p2, wt.data(), wt.size() * 8, hipMemcpyHostToDevice) != hipSuccess ||
            hipMemcpy(p3, bb.data(), bb.size() * 8, hipMemcpyHostToDevice) != hipSuccess) {
            leb_mlp_destroy(net);
            return LEB_EDEVICE;
        }
        net->W[l] = (double*)p1; net->WT[l] = (double*)p2; net->b[l] = (double*)p3;
    }
    *out = net;
    return LEB_OK;
}

extern "C" int leb_mlp_destroy(leb_mlp net) {
    if (!net) return LEB_OK;
    for (void* p : net->allocs) (void)hipFree(p);
    delete net;
    return LEB_OK;
}

namespace leb {

void nn_dims(const leb_mlp_s* net, int* nx, int* nu, int* m) {
    *nx = net->nx;
    *nu = net->nu;
    *m = net->w[net->L];
}

// Sizes (bytes) of the 21 work buffers of the bound for chunks of CB boxes.
void nn_buffer_sizes(const leb_mlp_s* net, int CB, size_t sizes[NN_NBUF]) {
    const int L = net->L, n0 = net->w[0], m = net->w[L];
    const size_t per = (size_t)CB * NN_MAXW * 8;
    const size_t lam = (size_t)CB * 3 * NN_MAXW * n0 * 8;          // Lambda_0 of every row, mode and box
    const size_t v3 = (size_t)CB * 3 * NN_MAXW * 8;
    const size_t tab[NN_NBUF] = {(size_t)CB * n0 * 8, (size_t)CB * n0 * 8, (size_t)CB * n0 * 8, per * (L - 1),
                                 per * (L - 1), per * (L - 1), (size_t)CB * m * 8, (size_t)CB * m * 8,
                                 per * (L - 1), per * (L - 1), per * (L - 1), per * (L - 1), per * (L - 1),
                                 per * (L - 1), lam, 8, v3, v3, v3, v3, (size_t)CB * 8};
    for (int q = 0; q < NN_NBUF; ++q) sizes[q] = tab[q];
}

// The bound of `units` boxes in chunks of CB, with caller-provided work
// buffers (nn_buffer_sizes); only kernels are enqueued on st.
int nn_bound_run(const leb_mlp_s* net, int64_t units, const double* z, const double* v, const double* mu,
                 const double* sigma, const double* J, double* r_lo, double* r_hi, double* c_bar, double* rho_bar,
                 double pad, uint32_t* flags, int CB, double* const* buf, hipStream_t st) {
    const int L = net->L, n0 = net->w[0], m = net->w[L];
    int rc;
    double *alpha = buf[0], *c = buf[1], *rho = buf[2], *zhat = buf[3], *lo = buf[4], *hi = buf[5], *g = buf[6],
           *eg = buf[7], *s = buf[8], *t = buf[9], *a = buf[10], *D = buf[11], *e = buf[12], *amax = buf[13],
           *bufA = buf[14], *beta = buf[16], *eps = buf[17];
    uint32_t* fl = (uint32_t*)buf[20];
    auto layer = [&](double* base, int l) { return base + (size_t)l * CB * NN_MAXW; };   // hidden layer l+1

    for (int64_t u0 = 0; u0 < units; u0 += CB) {
        const int nb = (int)((units - u0) < CB ? (units - u0) : CB);
        PrepArgs pa;
        pa.z = z; pa.v = v; pa.mu = mu; pa.sigma = sigma; pa.u0 = u0; pa.nbox = CB; pa.nact = nb;
        pa.L = L;
        for (int l = 0; l <= L; ++l) pa.w[l] = net->w[l];
        pa.nx = net->nx; pa.nu = net->nu;
        for (int l = 0; l < L; ++l) { pa.W[l] = net->W[l]; pa.WT[l] = net->WT[l]; pa.b[l] = net->b[l]; }
        pa.alpha = alpha; pa.c = c; pa.rho = rho; pa.zhat = zhat; pa.lo = lo; pa.hi = hi; pa.g = g; pa.eg = eg;
        pa.flags = fl;
        pa.s = s; pa.t = t; pa.a = a; pa.D = D; pa.e = e; pa.amax = amax;
        const bool groups = nb >= NNG_MIN;
        const int ng = (nb + NNG_BOXES - 1) / NNG_BOXES;
        if (groups) {
            static DynLds lds;
            if ((rc = lds.raise((const void*)nn_prep_group_kernel, NNG_LDS))) return rc;
            hipLaunchKernelGGL(nn_prep_group_kernel, dim3(ng), dim3(NNG_T), NNG_LDS, st, pa);
        } else {
            hipLaunchKernelGGL(nn_prep_kernel, dim3(nb), dim3(256), 0, st, pa);
        }
        if (hipGetLastError() != hipSuccess) return LEB_EDEVICE;
        auto relax = [&](int l) -> int {     // hidden layer l+1 (0-based l >= 1)
            RelaxArgs ra;
            ra.lo = layer(lo, l); ra.hi = layer(hi, l);
            ra.amax_prev = layer(amax, l - 1);
            ra.WT = net->WT[l]; ra.b = net->b[l]; ra.zhat = layer(zhat, l);
            ra.in = net->w[l]; ra.out = net->w[l + 1];
            ra.s = layer(s, l); ra.t = layer(t, l); ra.a = layer(a, l); ra.D = layer(D, l);
            ra.e = layer(e, l); ra.amax = layer(amax, l);
            ra.boxflags = fl;
            ra.nact = nb;
            if (groups) hipLaunchKernelGGL(nn_relax_group_kernel, dim3(ng), dim3(NNG_T), 0, st, ra);
            else hipLaunchKernelGGL(nn_relax_kernel, dim3(nb), dim3(256), 0, st, ra);
            return hipGetLastError() == hipSuccess ? LEB_OK : LEB_EDEVICE;
        };
        // backward chain for target layer k (1-based, 2..L): modes 0 upper, 1 lower (, 2 Jacobian)
        auto chain = [&](int k, int nmode, double** lam_out, double** beta_out, double** eps_out) -> int {
            ChainArgs ca = {};
            ca.WTt = net->WT[k - 1]; ca.bt = net->b[k - 1];
            for (int l = 0; l < L; ++l) { ca.W[l] = net->W[l]; ca.b[l] = net->b[l]; }
            for (int l = 0; l <= L; ++l) ca.w[l] = net->w[l];
            ca.k = k; ca.M = net->w[k]; ca.nbox = CB;
            ca.s = s; ca.t = t; ca.a = a; ca.D = D; ca.e = e; ca.lo = lo; ca.hi = hi;
            ca.bstride = ca.dbstride = NN_MAXW; ca.lstride = ca.dlstride = (size_t)CB * NN_MAXW;
            ca.C = bufA; ca.beta = beta; ca.eps = eps;
            if ((rc = launch_nn_chain<false>(ca, nmode, nb, st))) return rc;
            *lam_out = bufA; *beta_out = beta; *eps_out = eps;
            return LEB_OK;
        };
        for (int k = 2; k <= L - 1; ++k) {
            if (n0 == 16 && k <= 3) {
                // one or two steps down to a 16-wide input (one MFMA tile): both modes and the
                // concretisation in one launch (3,200 boxes of 16-256-256-256-12: 1.5 ms for the
                // two targets, 5.0 ms by the general chain); deeper targets and other inputs below
                HidArgs ha = {};
                ha.WTt = net->WT[k - 1]; ha.bt = net->b[k - 1];
                ha.W1 = net->W[0]; ha.b1 = net->b[0]; ha.W2 = net->W[1]; ha.b2 = net->b[1];
                ha.w1 = net->w[1]; ha.w2 = net->w[2]; ha.M = net->w[k];
                ha.s = s; ha.t = t; ha.a = a; ha.e = e; ha.lo = lo; ha.hi = hi;
                ha.bstride = NN_MAXW; ha.lstride = (size_t)CB * NN_MAXW;
                ha.c = c; ha.rho = rho; ha.cstride = 16;
                ha.lo_out = layer(lo, k - 1); ha.hi_out = layer(hi, k - 1);
                if (k == 2) hipLaunchKernelGGL(nn_hid1_kernel<false>, dim3(nb), dim3(256), 0, st, ha);
                else hipLaunchKernelGGL(nn_hid2_kernel<false>, dim3((ha.M + 31) / 32, nb), dim3(256), 0, st, ha);
                if (hipGetLastError() != hipSuccess) return LEB_EDEVICE;
                if ((rc = relax(k - 1))) return rc;
                continue;
            }
            double *L0, *bt, *ep;
            if ((rc = chain(k, 2, &L0, &bt, &ep))) return rc;
            ConcArgs ca;
            ca.L0 = L0; ca.beta = bt; ca.eps = ep; ca.c = c; ca.rho = rho;
            ca.M = net->w[k]; ca.n0 = n0; ca.nbox = CB;
            ca.lo = layer(lo, k - 1); ca.hi = layer(hi, k - 1);
            hipLaunchKernelGGL(nn_concretize_kernel, dim3(nb, 2), dim3(256), 0, st, ca);
            if (hipGetLastError() != hipSuccess) return LEB_EDEVICE;
            if ((rc = relax(k - 1))) return rc;
        }
        double *L0, *bt, *ep;
        // the Jacobian chain (mode 2) only when the caller gives no J
        if ((rc = chain(L, J ? 2 : 3, &L0, &bt, &ep))) return rc;
        Thm2Args ta;
        ta.L0 = L0; ta.beta = bt; ta.eps = ep; ta.alpha = alpha; ta.c = c; ta.rho = rho; ta.g = g; ta.eg = eg;
        ta.flags = fl; ta.Juser = J; ta.m = m; ta.n0 = n0; ta.nbox = CB; ta.u0 = u0;
        ta.r_lo = r_lo; ta.r_hi = r_hi; ta.c_bar = c_bar; ta.rho_bar = rho_bar; ta.pad = pad; ta.flags_out = flags;
        hipLaunchKernelGGL(nn_thm2_kernel, dim3(nb), dim3(64), 0, st, ta);
        if (hipGetLastError() != hipSuccess) return LEB_EDEVICE;
    }
    return LEB_OK;
}

}  // namespace leb

extern "C" int leb_nn_bound(leb_mlp net, int32_t batch, int32_t N, const double* z, const double* v, const double* mu,
                            const double* sigma, const double* J, double* r_lo, double* r_hi, double* c_bar,
                            double* rho_bar, double pad, uint32_t* flags, void* stream) {
    if (!net) return LEB_EINVAL;
    if (batch < 0 || N < 0 || !(pad >= 0.0) || !isfinite(pad)) return LEB_EINVAL;
    if ((c_bar == nullptr) != (rho_bar == nullptr)) return LEB_EINVAL;
    const int64_t units = (int64_t)batch * N;
    if (units == 0) return LEB_OK;
    if (!z || !sigma || !r_lo || !r_hi || (net->nu > 0 && !v) || (net->nx > 0 && !z)) return LEB_EINVAL;
    const void* ptrs[] = {z, v, mu, sigma, J, r_lo, r_hi, c_bar, rho_bar};
    for (const void* p : ptrs)
        if (p && !aligned8(p)) return LEB_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    const int L = net->L, n0 = net->w[0], m = net->w[L];
    std::lock_guard<std::mutex> lock(g_nnws.mu);
    const int CB = (int)(units < NN_CHUNK ? units : NN_CHUNK);
    size_t sizes[NN_NBUF];
    nn_buffer_sizes(net, CB, sizes);
    double* buf[NN_NBUF];
    int rc;
    for (int q = 0; q < NN_NBUF; ++q)
        if ((rc = nn_ws(q, sizes[q], &buf[q]))) return rc;
    if ((rc = g_nnws.fence.enter(st))) return rc;
    WsFenceScope leave{g_nnws.fence, st};
    return nn_bound_run(net, units, z, v, mu, sigma, J, r_lo, r_hi, c_bar, rho_bar, pad, flags, CB, buf, st);
}
