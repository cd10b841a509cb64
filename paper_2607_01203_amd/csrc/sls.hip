// sls.hip -- the system-level-synthesis layer around the bound: closed-loop
// responses from the parallel Riccati recursions, the time-varying tube map
// over them, the state-dependent disturbance error, and the exact tube/LEB
// fixed point of one controller update.
//
// Responses (appendix on solving for Phi, eqs. backward_prop and
// forward_prop; reformulated problem eq. fastsls_qp_reform): the problem
// splits over the disturbance time j, so every (trajectory, j) pair runs on its
// own, by one of two kernels chosen by size (leb_sls_responses),
//   backward  P_{N,j} = diag(qx_{N,j}); for k = N-1 .. j+1:
//             S = diag(qu_{k,j}) + B_k^T P B_k,  Bc = B_k^T P A_k,
//             K_{k,j} = -S^-1 Bc,  P <- diag(qx_{k,j}) + A_k^T P A_k + K^T Bc
//   forward   X = I; for k = j+1 .. N-1: Phi^x_{k,j} = X, Phi^u_{k,j} = K_{k,j} X,
//             X <- (A_k + B_k K_{k,j}) X.
// All FP64: the gains define the controller, they are not enclosures.
//
// Tube (eqs. tight_tube_center, tight_tube_width) with per-step disturbance
// matrices E_j [nx][nw]:
//   mu_k = sum_{j<k} Phi_{k,j} c_bar_j,
//   sigma_k = sum_{j<k} |Phi_{k,j} E_j| 1 + |Phi_{k,j}| rho_bar_j,
// plus an allowance that covers the FP64 rounding of both sums.  The blocks
// Phi_{k,0..k-1} of one row k are contiguous, so a workgroup streams its row
// once, coalesced, through LDS.
//
// Fixed point (section V loop, Theorem 3): the map from the bounds to the
// tube is causal (the tube at k needs the bounds at j < k only), so one pass
// over k in order gives the exact fixed point C = F(C): step k runs one row
// launch (finish step k-1's residual zonotope, then the tube row k) and one
// bound launch over all trajectories at step k.  The tube rows round upward
// and the bounds are outward, so C is a post-fixed point of the exact map and
// the Theorem 3 induction holds.
//
// Disturbance error (eqs. linearization_error_dist, interval_r_dist): with a
// thrust-magnitude disturbance of every planar quadrotor of a chain (total
// thrust (u1 + u2) + thrust w_i), node i's column of E(x) is
// thrust dt/m (-sin theta_i, cos theta_i) on its (vx, vz) rows; over the tube
// set, r_dist lies in +-s with s = mag([E](Omega^x_k) - E_k) row-summed.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>

#include "dpp.hpp"
#include "leb.h"
#include "leb_internal.hpp"
#include "pbh_node.hpp"

namespace leb {

constexpr int SLS_MAX_NX = 32;
constexpr int SLS_MAX_NU = 16;
constexpr int SLS_MAX_NW = 64;
constexpr int SLS_THREADS = 256;
constexpr size_t SLS_ROW_LDS = 48 * 1024;      // LDS budget of a tube-row workgroup
constexpr size_t SLS_LDS_MAX = 160 * 1024;     // LDS of the one-launch fixed point (a compute unit's)

// ------------------------------------------------------------ responses

struct RiccatiArgs {
    const double* A; const double* B; const double* qx; const double* qu;
    double* K; double* phi;
    int nx, nu, N;
    int zero;                // 1: write 0 to the entries k <= j too
};

// Zeros of disturbance times j .. j + cnt - 1 (adjacent in memory), every k <= j: the
// workgroup's last work.  A chain has j + 1 blocks to clear and N - j - 1 steps to run,
// so the clearing fills the memory system while the long chains still run (as a fill of
// the whole arrays before the launch it cost 25 us at 256 x 40, nx = 6, and 0.25 ms at
// 64 x 40, nx = 30).
__device__ void riccati_zero(const RiccatiArgs& a, int b, int j, int cnt) {
    const int nk = a.nu * a.nx, np = (a.nx + a.nu) * a.nx;
    const int last = min(j + cnt, a.N) - 1;
    for (int k = 0; k <= last; ++k) {
        const int j0 = max(j, k);                 // times j0 .. last have k <= j
        const size_t o = ((size_t)b * a.N + k) * a.N + j0;
        double* K = a.K + o * nk;
        double* P = a.phi + o * np;
        const int m = last - j0 + 1;
        for (int q = threadIdx.x; q < m * nk; q += blockDim.x) K[q] = 0.0;
        for (int q = threadIdx.x; q < m * np; q += blockDim.x) P[q] = 0.0;
    }
}

// One small size (NX <= 8, NU = 2) with eight lanes per
// (trajectory, j): lane c of a group of eight holds column c of every matrix in
// registers, so products with A_k and B_k from the left are local, and a wave
// runs eight consecutive j of one trajectory in lockstep over k, sharing
// A_k and B_k (read as broadcasts from LDS, stored there one step ahead).
// P is symmetric, so P A = (A^T P)^T: the step's only exchanges between lanes are
// that transpose, the 2 x NX rows of B^T P, the gain and P's own transpose (LDS, padded
// strides).  As in the tiled kernel below, P is made symmetric, here after every second step:
// 99th percentile of the gains' relative error against long double, 40 steps of the hover
// workload, 1.4e-15, with weights 1e4 apart 2.4e-15 (after each step 1.4e-15 and 2.1e-15
// at 7 us more; after every eighth 1.9e-15 and 1.9e-14; P as it comes 4.2e-14 and 4.8e-12).
// The 2 x 2 system is solved as L D L^T; its pivots are the squares of the
// Cholesky pivots and are tested the same way.
//
// What bounds it: the serial chain of a wave, 2 (N - j - 1) dependent steps; at
// 256 trajectories a compute unit holds five waves.  Eight lanes per chain keep
// one step's products (about 190 FMA) inside the latency that its exchanges cost
// anyway.  256 x 40 steps at nx = 6: 0.089 ms (0.085 without the means of P; one 64-lane
// workgroup per chain with the matrices in LDS: 0.280 ms); 1,024 x 40: 0.24 ms (0.857 ms).
template <int NX, int NU>
__global__ void __launch_bounds__(64) sls_riccati_lane_kernel(RiccatiArgs a) {
    static_assert(NX <= 8 && NU == 2, "eight lanes per chain, 2 x 2 gain system");
    constexpr int n = NX + NU, AB = NX * n;                    // A_k and B_k of one step
    constexpr int ST = NX * NX + 2, SN = NU * NX + 2;          // strides of a chain's blocks in LDS
    constexpr int SYM = 2;                                     // steps from one mean of P to the next
    const int b = blockIdx.y, N = a.N;
    const int lane = threadIdx.x, ch = lane >> 3, c = lane & 7;
    const int j0 = 8 * blockIdx.x, j = min(j0 + ch, N - 1);   // j = N - 1 has no steps
    const bool own = c < NX;
    const int cc = own ? c : 0;
    __shared__ double sAB[2][AB];
    __shared__ double sT[8 * ST];                              // A^T P, then free
    __shared__ double sN[8 * SN];                              // B^T P, then K
    const double* Ab = a.A + (size_t)b * N * NX * NX;
    const double* Bb = a.B + (size_t)b * N * NX * NU;
    const double* qxb = a.qx + (size_t)b * (N + 1) * N * NX;
    const double* qub = a.qu + (size_t)b * N * N * NU;
    double* Kb = a.K + (size_t)b * N * N * NU * NX;
    double* phib = a.phi + (size_t)b * N * N * n * NX;
    auto ab_at = [&](int k) {
        return lane < NX * NX ? Ab[(size_t)k * NX * NX + lane]
                              : (lane < AB ? Bb[(size_t)k * NX * NU + (lane - NX * NX)] : 0.0);
    };
    static_assert(AB <= 64, "one value of A_k and B_k per lane");
    double P[NX];
#pragma unroll
    for (int r = 0; r < NX; ++r) P[r] = 0.0;
    {
        const double q = qxb[((size_t)N * N + j) * NX + cc];
#pragma unroll
        for (int r = 0; r < NX; ++r) P[r] = r == c ? q : 0.0;
    }
    double abn = ab_at(N - 1);
    double qxn = qxb[((size_t)(N - 1) * N + j) * NX + cc];
    double qu0n = qub[((size_t)(N - 1) * N + j) * NU], qu1n = qub[((size_t)(N - 1) * N + j) * NU + 1];
    if (lane < AB) sAB[(N - 1) & 1][lane] = abn;
    if (N - 2 > j0) abn = ab_at(N - 2);
    for (int k = N - 1; k > j0; --k) {
        const double qx = qxn, qu0 = qu0n, qu1 = qu1n;
        lds_barrier();                                         // A_k, B_k stored; sN free
        if (k - 1 > j0) {
            qxn = qxb[((size_t)(k - 1) * N + j) * NX + cc];
            qu0n = qub[((size_t)(k - 1) * N + j) * NU];
            qu1n = qub[((size_t)(k - 1) * N + j) * NU + 1];
        }
        double A[NX * NX], B[NX * NU];
#pragma unroll
        for (int q = 0; q < NX * NX; ++q) A[q] = sAB[k & 1][q];
#pragma unroll
        for (int q = 0; q < NX * NU; ++q) B[q] = sAB[k & 1][NX * NX + q];
        // column c of A^T P (row c of P A) and of B^T P
#pragma unroll
        for (int r = 0; r < NX; ++r) {
            double s = 0.0;
#pragma unroll
            for (int l = 0; l < NX; ++l) s = fma(A[l * NX + r], P[l], s);
            if (own) sT[ch * ST + c * NX + r] = s;
        }
#pragma unroll
        for (int m = 0; m < NU; ++m) {
            double s = 0.0;
#pragma unroll
            for (int l = 0; l < NX; ++l) s = fma(B[l * NU + m], P[l], s);
            if (own) sN[ch * SN + m * NX + c] = s;
        }
        lds_barrier();
        if (k - 1 > j0) {
            if (lane < AB) sAB[(k - 1) & 1][lane] = abn;
            if (k - 2 > j0) abn = ab_at(k - 2);
        }
        double PA[NX], Bc[NU], S[3];                           // S: (0,0), (1,0), (1,1)
#pragma unroll
        for (int r = 0; r < NX; ++r) PA[r] = sT[ch * ST + r * NX + cc];
        S[0] = S[1] = S[2] = 0.0;
#pragma unroll
        for (int l = 0; l < NX; ++l) {
            const double n0 = sN[ch * SN + l], n1 = sN[ch * SN + NX + l];
            S[0] = fma(n0, B[l * NU], S[0]);
            S[1] = fma(n1, B[l * NU], S[1]);
            S[2] = fma(n1, B[l * NU + 1], S[2]);
        }
#pragma unroll
        for (int m = 0; m < NU; ++m) {
            Bc[m] = 0.0;
#pragma unroll
            for (int r = 0; r < NX; ++r) Bc[m] = fma(B[r * NU + m], PA[r], Bc[m]);
        }
        double d0 = qu0 + S[0];
        bool bad = !(d0 > 0.0) || !isfinite(d0);
        if (bad) d0 = 1.0;
        const double i0 = 1.0 / d0, l10 = S[1] * i0;
        double d1 = fma(-l10, S[1], qu1 + S[2]);
        if (!(d1 > 0.0) || !isfinite(d1)) { bad = true; d1 = 1.0; }
        const double y1 = fma(-l10, Bc[0], Bc[1]) / d1;
        const double y0 = fma(-l10, y1, Bc[0] * i0);
        const double K0 = bad ? NAN : -y0, K1 = bad ? NAN : -y1;
        lds_barrier();                                         // B^T P read
        if (own) {
            sN[ch * SN + c] = K0;
            sN[ch * SN + NX + c] = K1;
            if (k > j) {
                double* Kp = Kb + ((size_t)k * N + j) * NU * NX;
                Kp[c] = K0;
                Kp[NX + c] = K1;
            }
        }
        lds_barrier();
        // P <- diag(qx) + A^T (P A) + K^T Bc (chains with k <= j no longer use theirs)
#pragma unroll
        for (int r = 0; r < NX; ++r) {
            double s = r == c ? qx : 0.0;
#pragma unroll
            for (int l = 0; l < NX; ++l) s = fma(A[l * NX + r], PA[l], s);
            s = fma(sN[ch * SN + r], Bc[0], s);
            P[r] = fma(sN[ch * SN + NX + r], Bc[1], s);
        }
        if ((k & (SYM - 1)) == 0) {
            // the mean with the transpose (element (c, r) is in lane r's column)
#pragma unroll
            for (int r = 0; r < NX; ++r)
                if (own) sT[ch * ST + c * NX + r] = P[r];
            lds_barrier();
#pragma unroll
            for (int r = 0; r < NX; ++r) P[r] = 0.5 * (P[r] + sT[ch * ST + r * NX + cc]);
        }
    }
    // forward: U = K X, X' = A X + B U from Phi^x_{j+1,j} = I.  The gains were stored
    // by this wave, and the full barrier orders those stores before the loads
    __syncthreads();
    double X[NX], Kn[NU * NX];
#pragma unroll
    for (int r = 0; r < NX; ++r) X[r] = 0.0;
    auto kfetch = [&](int k) {
        const double* Kp = Kb + ((size_t)k * N + min(j, k - 1)) * NU * NX;
#pragma unroll
        for (int q = 0; q < NU * NX; ++q) Kn[q] = Kp[q];
    };
    abn = ab_at(j0 + 1 < N ? j0 + 1 : N - 1);
    if (j0 + 1 < N) {
        kfetch(j0 + 1);
        if (lane < AB) sAB[(j0 + 1) & 1][lane] = abn;
        if (j0 + 2 < N) abn = ab_at(j0 + 2);
    }
    for (int k = j0 + 1; k < N; ++k) {
        double K[NU * NX];
#pragma unroll
        for (int q = 0; q < NU * NX; ++q) K[q] = Kn[q];
        lds_barrier();                                         // A_k, B_k stored
        if (k + 1 < N) kfetch(k + 1);
        if (k == j + 1) {
#pragma unroll
            for (int r = 0; r < NX; ++r) X[r] = r == c ? 1.0 : 0.0;
        }
        double U[NU];
#pragma unroll
        for (int m = 0; m < NU; ++m) {
            U[m] = 0.0;
#pragma unroll
            for (int l = 0; l < NX; ++l) U[m] = fma(K[m * NX + l], X[l], U[m]);
        }
        if (own && k > j) {
            double* out = phib + ((size_t)k * N + j) * n * NX + c;
#pragma unroll
            for (int r = 0; r < NX; ++r) out[r * NX] = X[r];
#pragma unroll
            for (int m = 0; m < NU; ++m) out[(NX + m) * NX] = U[m];
        }
        double Xn[NX];
#pragma unroll
        for (int r = 0; r < NX; ++r) {
            double s = 0.0;
#pragma unroll
            for (int l = 0; l < NX; ++l) s = fma(sAB[k & 1][r * NX + l], X[l], s);
#pragma unroll
            for (int m = 0; m < NU; ++m) s = fma(sAB[k & 1][NX * NX + r * NU + m], U[m], s);
            Xn[r] = s;
        }
#pragma unroll
        for (int r = 0; r < NX; ++r) X[r] = Xn[r];
        if (k + 1 < N) {
            if (lane < AB) sAB[(k + 1) & 1][lane] = abn;
            if (k + 2 < N) abn = ab_at(k + 2);
        }
    }
    if (a.zero) riccati_zero(a, b, j0, 8);
}

typedef double sls_d4 __attribute__((ext_vector_type(4)));

// Every other size (nx <= 32, nu <= 16) on FP64 MFMA (v_mfma_f64_16x16x4f64): one
// wave per (trajectory, j), every matrix in registers as TX x TX zero-padded
// 16 x 16 tiles (TX = 2: nx > 16) in the accumulator layout (lane l holds element
// [4i + l/16][l%16] of its tile, i = 0..3).  That layout is also the B operand of a
// product and, read as the A operand, the transpose, so every product is a sum of
// X^T Y over tiles and stays in registers:
//   P A = P^T A and P B = P^T B (P is symmetric), S = B^T (P B),
//   Bc = B^T (P A), P' = diag(qx) + A^T (P A) + K^T Bc;
//   forward: U = (K^T)^T X, X' = (A^T)^T X + (B^T)^T U,
// with A^T, B^T, K^T loaded straight into the layout.  The gain solves S K = -Bc by elimination: lane c
// holds column c of [S | Bc] (NUB rows, NUB >= nu), and the pivot column is read
// from its lane by v_readlane, so the nu steps need no LDS; the pivots are
// the squares of the Cholesky pivots' and are tested the same way.  Only the
// hand-over between the two layouts goes through LDS.
//
// P is made symmetric after each step (the mean with its transpose, through LDS):
// the products take P for its transpose, and the antisymmetric part of P's rounding
// grows along the chain.  99th percentile of the gains' relative error against long
// double, 40 steps, nx = 30: 2.0e-15, and 9.9e-13 with weights 1e4 apart (every
// matrix in LDS, P as it comes: 7.8e-14 and 2.4e-12).
//
// What bounds it: the FP64 matrix rate and the serial chain of a wave.  At
// nx = 30, nu = 10 a backward and a forward step issue 184 MFMA (64 cycles
// each); the first launched waves are the longest chains (j = 0 of every
// trajectory), so the short ones fill the end of the launch.  64 x 40 steps:
// 0.61 ms, 29 TFLOP/s of padded products (6.48 ms with a 256-lane workgroup per
// (trajectory, j) and every matrix in LDS).  Small sizes too: 256 x 40 steps at
// nx = 12, nu = 4: 0.31 ms (0.55 ms with whole tiles multiplied and every lane
// factoring S); at nx = 8, nu = 4: 0.30 ms and at nx = 1: 0.19 ms (0.60 and 0.30 ms
// with the matrices in LDS on the VALU).
// Tiles are read through a buffer descriptor of the one matrix: a row past the
// end is out of its range and reads 0, so a lane needs one offset per tile and one
// column test instead of an address and a test for every element.
typedef unsigned int sls_u2 __attribute__((ext_vector_type(2)));
typedef unsigned int sls_u4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t matrix_rsrc(const double* M, int elems) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(M), 0, elems * 8, 0x00027000);
}

// the 16 x 16 tile at (r0, c0) of a matrix with rows of C elements; tr: of its transpose
__device__ __forceinline__ sls_d4 tile_at(__amdgpu_buffer_rsrc_t M, int C, int r0, int c0, int lr, int lq, bool tr) {
    sls_d4 v;
    const int o = 8 * (tr ? (c0 + lr) * C + r0 + lq : (r0 + lq) * C + c0 + lr);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        union { sls_u2 u; double d; } x;
        x.u = __builtin_amdgcn_raw_buffer_load_b64(M, o + (tr ? 32 * i : 32 * i * C), 0, 0);
        v[i] = (tr ? r0 + lq + 4 * i : c0 + lr) < C ? x.d : 0.0;
    }
    return v;
}

__device__ __forceinline__ double lane_value(double x, int lane) {   // x of one lane, uniform
    union { double d; int w[2]; } u;
    u.d = x;
    u.w[0] = __builtin_amdgcn_readlane(u.w[0], lane);
    u.w[1] = __builtin_amdgcn_readlane(u.w[1], lane);
    return u.d;
}

// acc + X^T Y over the first `steps` groups of four rows (the others are padding)
__device__ __forceinline__ sls_d4 mm_tn(const sls_d4& X, const sls_d4& Y, sls_d4 acc, int steps) {
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[0], Y[0], acc, 0, 0, 0);
    if (steps > 1) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[1], Y[1], acc, 0, 0, 0);
    if (steps > 2) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[2], Y[2], acc, 0, 0, 0);
    if (steps > 3) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[3], Y[3], acc, 0, 0, 0);
    return acc;
}

template <int TX, int NUB>
__global__ void __launch_bounds__(64, 2) sls_riccati_tile_kernel(RiccatiArgs a) {
    constexpr int W = 16 * TX, LD = 16 + W;
    const int b = blockIdx.x, j = blockIdx.y;
    const int nx = a.nx, nu = a.nu, N = a.N, n = nx + nu;
    if (j >= N - 1) {                            // no k with j < k < N
        if (a.zero) riccati_zero(a, b, j, 1);
        return;
    }
    // k-steps of a product over states (per tile) and over inputs
    const int sx0 = TX > 1 ? 4 : (nx + 3) >> 2, sx1 = (nx - 13) >> 2, su = (nu + 3) >> 2;
    auto sx = [&](int t) { return t == 0 ? sx0 : sx1; };
    __shared__ double sT[16 * LD];               // [S | Bc], row-major
    __shared__ double sK[16 * W];                // K_k, zero rows past nu
    __shared__ double sP[W * (W + 1)];           // P, to be read transposed
    const int lane = threadIdx.x, lr = lane & 15, lq = lane >> 4;
    const double* Ab = a.A + (size_t)b * N * nx * nx;
    const double* Bb = a.B + (size_t)b * N * nx * nu;
    const double* qxb = a.qx + (size_t)b * (N + 1) * N * nx;
    const double* qub = a.qu + (size_t)b * N * N * nu;
    double* Kb = a.K + (size_t)b * N * N * nu * nx;
    double* phib = a.phi + (size_t)b * N * N * n * nx;
    for (int q = lane; q < 16 * W; q += 64) sK[q] = 0.0;
    // element of this lane on a tile's diagonal (row 4i + lq == lr), if any
    const int di = (lr >= lq && ((lr - lq) & 3) == 0) ? (lr - lq) >> 2 : -1;
    const sls_d4 z4 = {0.0, 0.0, 0.0, 0.0};
    auto diag = [&](const double* q, int t) { return (di >= 0 && 16 * t + lr < nx) ? q[16 * t + lr] : 0.0; };
    sls_d4 P[TX][TX], An[TX][TX], Bn[TX];
    double qxn[TX], qun;
#pragma unroll
    for (int t = 0; t < TX; ++t) {
        const double q = diag(qxb + ((size_t)N * N + j) * nx, t);
#pragma unroll
        for (int u = 0; u < TX; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) P[t][u][i] = (t == u && i == di) ? q : 0.0;
    }
    auto fetch = [&](int k) {
        const auto rA = matrix_rsrc(Ab + (size_t)k * nx * nx, nx * nx), rB = matrix_rsrc(Bb + (size_t)k * nx * nu, nx * nu);
#pragma unroll
        for (int t = 0; t < TX; ++t) {
#pragma unroll
            for (int u = 0; u < TX; ++u) An[t][u] = tile_at(rA, nx, 16 * t, 16 * u, lr, lq, false);
            Bn[t] = tile_at(rB, nu, 16 * t, 0, lr, lq, false);
            qxn[t] = diag(qxb + ((size_t)k * N + j) * nx, t);
        }
        qun = (di >= 0 && lr < nu) ? qub[((size_t)k * N + j) * nu + lr] : 0.0;
    };
    fetch(N - 1);
    for (int k = N - 1; k > j; --k) {
        sls_d4 A[TX][TX], B[TX], PA[TX][TX], Bc[TX];
        double qxd[TX];
        const double qud = qun;
#pragma unroll
        for (int t = 0; t < TX; ++t) {
#pragma unroll
            for (int u = 0; u < TX; ++u) A[t][u] = An[t][u];
            B[t] = Bn[t];
            qxd[t] = qxn[t];
        }
        if (k - 1 > j) fetch(k - 1);
        // S = diag(qu) + B^T (P B) first: its elimination is the longer chain
        sls_d4 S = z4;
#pragma unroll
        for (int t = 0; t < TX; ++t) {
            sls_d4 pb = z4;
#pragma unroll
            for (int u = 0; u < TX; ++u) pb = mm_tn(P[u][t], B[u], pb, sx(u));
            S = mm_tn(B[t], pb, S, sx(t));
        }
#pragma unroll
        for (int t = 0; t < TX; ++t)
#pragma unroll
            for (int u = 0; u < TX; ++u) {
                sls_d4 c = z4;
#pragma unroll
                for (int l = 0; l < TX; ++l) c = mm_tn(P[l][t], A[l][u], c, sx(l));
                PA[t][u] = c;
            }
#pragma unroll
        for (int u = 0; u < TX; ++u) {
            Bc[u] = z4;
#pragma unroll
            for (int t = 0; t < TX; ++t) Bc[u] = mm_tn(B[t], PA[t][u], Bc[u], sx(t));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 4 * i + lq;
            sT[row * LD + lr] = S[i] + (i == di ? qud : 0.0);
#pragma unroll
            for (int u = 0; u < TX; ++u) sT[row * LD + 16 + 16 * u + lr] = Bc[u][i];
        }
        lds_barrier();
        // elimination: column `lane` of [S | Bc]
        {
            double col[NUB];
            const int c = lane < LD ? lane : LD - 1;
#pragma unroll
            for (int r = 0; r < NUB; ++r) col[r] = sT[r * LD + c];
            bool bad = false;
#pragma unroll
            for (int p = 0; p < NUB; ++p) {
                if (p < nu) {
                    double piv = lane_value(col[p], p);
                    if (!(piv > 0.0) || !isfinite(piv)) { bad = true; piv = 1.0; }
                    const double x = col[p] / piv;
#pragma unroll
                    for (int r = 0; r < NUB; ++r)
                        if (r != p) col[r] = fma(-lane_value(col[r], p), x, col[r]);
                    col[p] = x;
                }
            }
            const int kc = lane - 16;
            if (kc >= 0 && kc < W) {
#pragma unroll
                for (int r = 0; r < NUB; ++r) {
                    if (r < nu) {
                        const double kv = bad ? NAN : -col[r];
                        sK[r * W + kc] = kv;
                        if (kc < nx) Kb[((size_t)k * N + j) * nu * nx + r * nx + kc] = kv;
                    }
                }
            }
        }
        lds_barrier();
        // P <- diag(qx) + A^T (P A) + K^T Bc
        sls_d4 K[TX];
#pragma unroll
        for (int t = 0; t < TX; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) K[t][i] = sK[(4 * i + lq) * W + 16 * t + lr];
#pragma unroll
        for (int t = 0; t < TX; ++t)
#pragma unroll
            for (int u = 0; u < TX; ++u) {
                sls_d4 c;
#pragma unroll
                for (int i = 0; i < 4; ++i) c[i] = (t == u && i == di) ? qxd[t] : 0.0;
#pragma unroll
                for (int l = 0; l < TX; ++l) c = mm_tn(A[l][t], PA[l][u], c, sx(l));
                P[t][u] = mm_tn(K[t], Bc[u], c, su);
#pragma unroll
                for (int i = 0; i < 4; ++i) sP[(16 * t + 4 * i + lq) * (W + 1) + 16 * u + lr] = P[t][u][i];
            }
        lds_barrier();                           // sT, sK are rewritten by the next step, sP two barriers on
#pragma unroll
        for (int t = 0; t < TX; ++t)
#pragma unroll
            for (int u = 0; u < TX; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    P[t][u][i] = 0.5 * (P[t][u][i] + sP[(16 * u + lr) * (W + 1) + 16 * t + 4 * i + lq]);
    }
    // forward: U = K X, X' = A X + B U.  The gains were stored by this wave, and the
    // full barrier orders those stores before the loads
    __syncthreads();
    sls_d4 X[TX][TX], ATn[TX][TX], BTn[TX], KTn[TX];
#pragma unroll
    for (int t = 0; t < TX; ++t)
#pragma unroll
        for (int u = 0; u < TX; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) X[t][u][i] = (t == u && i == di && 16 * t + lr < nx) ? 1.0 : 0.0;
    auto ffetch = [&](int k) {                   // tiles of A^T, B^T, K^T
        const auto rA = matrix_rsrc(Ab + (size_t)k * nx * nx, nx * nx), rB = matrix_rsrc(Bb + (size_t)k * nx * nu, nx * nu),
                   rK = matrix_rsrc(Kb + ((size_t)k * N + j) * nu * nx, nu * nx);
#pragma unroll
        for (int t = 0; t < TX; ++t) {
#pragma unroll
            for (int u = 0; u < TX; ++u) ATn[t][u] = tile_at(rA, nx, 16 * t, 16 * u, lr, lq, true);
            BTn[t] = tile_at(rB, nu, 0, 16 * t, lr, lq, true);
            KTn[t] = tile_at(rK, nx, 16 * t, 0, lr, lq, true);
        }
    };
    ffetch(j + 1);
    for (int k = j + 1; k < N; ++k) {
        sls_d4 AT[TX][TX], BT[TX], KT[TX], U[TX];
#pragma unroll
        for (int t = 0; t < TX; ++t) {
#pragma unroll
            for (int u = 0; u < TX; ++u) AT[t][u] = ATn[t][u];
            BT[t] = BTn[t];
            KT[t] = KTn[t];
        }
        if (k + 1 < N) ffetch(k + 1);
#pragma unroll
        for (int u = 0; u < TX; ++u) {
            U[u] = z4;
#pragma unroll
            for (int t = 0; t < TX; ++t) U[u] = mm_tn(KT[t], X[t][u], U[u], sx(t));
        }
        double* out = phib + ((size_t)k * N + j) * n * nx;
#pragma unroll
        for (int u = 0; u < TX; ++u) {
            const int col = 16 * u + lr;
            if (col < nx) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
#pragma unroll
                    for (int t = 0; t < TX; ++t) {
                        const int row = 16 * t + 4 * i + lq;
                        if (row < nx) out[row * nx + col] = X[t][u][i];
                    }
                    if (4 * i + lq < nu) out[(nx + 4 * i + lq) * nx + col] = U[u][i];
                }
            }
        }
        if (k + 1 < N) {
            sls_d4 Xn[TX][TX];
#pragma unroll
            for (int t = 0; t < TX; ++t)
#pragma unroll
                for (int u = 0; u < TX; ++u) {
                    sls_d4 c = mm_tn(BT[t], U[u], z4, su);
#pragma unroll
                    for (int l = 0; l < TX; ++l) c = mm_tn(AT[l][t], X[l][u], c, sx(l));
                    Xn[t][u] = c;
                }
#pragma unroll
            for (int t = 0; t < TX; ++t)
#pragma unroll
                for (int u = 0; u < TX; ++u) X[t][u] = Xn[t][u];
        }
    }
    if (a.zero) riccati_zero(a, b, j, 1);
}

template <int TX>
static void launch_riccati_tile(const RiccatiArgs& a, int batch, hipStream_t st) {
    const dim3 grid((unsigned)batch, (unsigned)a.N);
    if (a.nu <= 4) hipLaunchKernelGGL((sls_riccati_tile_kernel<TX, 4>), grid, dim3(64), 0, st, a);
    else if (a.nu <= 8) hipLaunchKernelGGL((sls_riccati_tile_kernel<TX, 8>), grid, dim3(64), 0, st, a);
    else if (a.nu <= 12) hipLaunchKernelGGL((sls_riccati_tile_kernel<TX, 12>), grid, dim3(64), 0, st, a);
    else hipLaunchKernelGGL((sls_riccati_tile_kernel<TX, 16>), grid, dim3(64), 0, st, a);
}

// ------------------------------------------------------------ tube rows

struct TubeRowArgs {
    const double* phi;       // [b][N][N][n][nx]
    const double* E;         // [b][N][nx][nw]
    const double* cbar;      // [b][N][nx]
    const double* rbar;      // [b][N][nx]
    double* mu;              // [b][N][n]
    double* sigma;           // [b][N][n]
    const double* sigE;      // [b][N][n] the disturbance part of sigma (ROW_NOE reads it)
    int nx, nu, nw, N, jc;
};

// What a tube row sums: both parts of eq. tight_tube_width (ROW_FULL), only
// the disturbance part sum_j |Phi_{k,j} E_j| 1, which does not depend on the
// bounds (ROW_E), or the centre and the residual part, adding the disturbance
// part from sigE (ROW_NOE).
constexpr int ROW_FULL = 0, ROW_E = 1, ROW_NOE = 2;

// One trajectory's operands of tube row k (generic pointers: global or LDS).
struct RowRef {
    const double* phi;       // Phi_{k,0} (the row block of k)
    const double* E;         // E_0 (ROW_FULL, ROW_E)
    const double* cb;        // c_bar_0 (ROW_FULL, ROW_NOE)
    const double* rb;        // rho_bar_0
    const double* sigE;      // the disturbance part of row k, n values (ROW_NOE)
};

__device__ __forceinline__ RowRef row_ref(const TubeRowArgs& a, int b, int k) {
    const int nx = a.nx, n = nx + a.nu, N = a.N;
    RowRef r;
    r.phi = a.phi + (((size_t)b * N + k) * N) * n * nx;
    r.E = a.E ? a.E + (size_t)b * N * nx * a.nw : nullptr;
    r.cb = a.cbar ? a.cbar + (size_t)b * N * nx : nullptr;
    r.rb = a.rbar ? a.rbar + (size_t)b * N * nx : nullptr;
    r.sigE = a.sigE ? a.sigE + ((size_t)b * N + k) * n : nullptr;
    return r;
}

// Tube row k of trajectory b.  Thread t = jj * n + i works on row i of
// Phi_{k, j0 + jj}, which it loads straight into registers (every entry of
// Phi is used by one thread only); E_j, |E_j| 1, c_bar_j and rho_bar_j are
// shared through LDS, jc disturbance times per chunk.  NXB >= nx is the
// register length of a row.  Leaves the row's (mu, sigma) in mo[], so[] (LDS,
// n entries) after the final barrier.
template <int MODE, int NXB>
__device__ void tube_row(const TubeRowArgs& a, const RowRef& rr, int k, double* sm, double* mo, double* so) {
    const int nx = a.nx, nw = a.nw, n = nx + a.nu, jc = a.jc;
    const int tid = threadIdx.x, nt = blockDim.x;
    const bool useE = MODE != ROW_NOE, useR = MODE != ROW_E;
    double* sE = sm;                                          // jc*nx*nw   (useE)
    double* se1 = sE + (useE ? (size_t)jc * nx * nw : 0);     // jc*nx      (useE)
    double* scb = se1 + (useE ? jc * nx : 0);                 // jc*nx      (useR)
    double* srb = scb + (useR ? jc * nx : 0);                 // jc*nx      (useR)
    double* red = srb + (useR ? jc * nx : 0);                 // 3*jc*n
    const int jj = tid / n, i = tid - jj * n;
    const bool act = jj < jc;
    double am = 0.0, as = 0.0, ag = 0.0;
    const double* prow = rr.phi;
    for (int j0 = 0; j0 < k; j0 += jc) {
        const int cnt = min(jc, k - j0);
        const bool mine = act && jj < cnt;
        double r[NXB];
        if (mine) {
            const double* src = prow + ((size_t)(j0 + jj) * n + i) * nx;
#pragma unroll
            for (int l = 0; l < NXB; ++l) r[l] = l < nx ? src[l] : 0.0;
        }
        if (useE) {
            const double* ep = rr.E + (size_t)j0 * nx * nw;
            for (int q = tid; q < cnt * nx * nw; q += nt) sE[q] = ep[q];
        }
        if (useR) {
            const size_t ro = (size_t)j0 * nx;
            for (int q = tid; q < cnt * nx; q += nt) { scb[q] = rr.cb[ro + q]; srb[q] = rr.rb[ro + q]; }
        }
        lds_barrier();
        if (useE) {
            for (int q = tid; q < cnt * nx; q += nt) {
                double t = 0.0;
                for (int w = 0; w < nw; ++w) t += fabs(sE[q * nw + w]);
                se1[q] = t;
            }
            lds_barrier();
        }
        if (mine) {
            double m = 0.0, s = 0.0, g = 0.0;
            if (useR) {
                const double* cb = scb + jj * nx;
                const double* rb = srb + jj * nx;
#pragma unroll
                for (int l = 0; l < NXB; ++l) {
                    if (l < nx) {
                        const double ap = fabs(r[l]);
                        m = fma(r[l], cb[l], m);
                        s = fma(ap, rb[l], s);
                        g = fma(ap, fabs(cb[l]) + rb[l], g);
                    }
                }
            }
            if (useE) {
                const double* e1 = se1 + jj * nx;
                const double* Ej = sE + (size_t)jj * nx * nw;
#pragma unroll
                for (int l = 0; l < NXB; ++l)
                    if (l < nx) g = fma(fabs(r[l]), e1[l], g);
                for (int w = 0; w < nw; ++w) {
                    double t = 0.0;
#pragma unroll
                    for (int l = 0; l < NXB; ++l)
                        if (l < nx) t = fma(r[l], Ej[l * nw + w], t);
                    s += fabs(t);
                }
            }
            am += m; as += s; ag += g;
        }
        lds_barrier();
    }
    // partial sums over the disturbance-time slots: within each wave by a
    // butterfly over the lanes of one row (when n divides the wave and every
    // lane holds a slot), then over the waves; otherwise slot by slot
    const bool wave_red = (64 % n == 0) && (jc * n == nt);
    if (wave_red) {
        double m = am, s_ = as, g = ag;
        for (int msk = n; msk < 64; msk <<= 1) {
            m += __shfl_xor(m, msk);
            s_ += __shfl_xor(s_, msk);
            g += __shfl_xor(g, msk);
        }
        const int lane = tid & 63, wv = tid >> 6;
        if (lane < n) { red[(3 * wv) * n + lane] = m; red[(3 * wv + 1) * n + lane] = s_; red[(3 * wv + 2) * n + lane] = g; }
    } else if (act) {
        red[jj * n + i] = am; red[(jc + jj) * n + i] = as; red[(2 * jc + jj) * n + i] = ag;
    }
    lds_barrier();
    if (tid < n) {
        double m = 0.0, s = 0.0, g = 0.0;
        if (wave_red) {
            for (int w = 0; w < nt / 64; ++w) { m += red[(3 * w) * n + tid]; s += red[(3 * w + 1) * n + tid]; g += red[(3 * w + 2) * n + tid]; }
        } else {
            for (int q = 0; q < jc; ++q) { m += red[q * n + tid]; s += red[(jc + q) * n + tid]; g += red[(2 * jc + q) * n + tid]; }
        }
        // rounding of the sums: at most nx + k (nw + 1) + jc additions deep, each
        // within 2^-53 of the magnitudes g; doubled for the centre's error and the
        // final additions
        const double coef = (double)(nx + k * (nw + 1) + jc + 8) * 0x1p-52;
        s = s + coef * g * (1.0 + 0x1p-50) + 0x1p-1000;
        if (MODE == ROW_NOE) {
            const double se = rr.sigE[tid];
            s = s + se;
            s = s + fabs(s) * 0x1p-52;
            if (!isfinite(se)) g = INFINITY;
        }
        if (!isfinite(g) || !isfinite(s)) { m = 0.0; s = INFINITY; }
        if (k == 0) { m = 0.0; s = 0.0; }
        mo[tid] = MODE == ROW_E ? 0.0 : m;
        so[tid] = s;
    }
    __syncthreads();
}

static int tube_jc(int nx, int nu, int nw, int mode, size_t* smem) {
    const int n = nx + nu;
    const size_t per_j = sizeof(double) * ((mode != ROW_NOE ? (size_t)nx * nw + nx : 0) +
                                           (mode != ROW_E ? 2 * (size_t)nx : 0) + 3 * (size_t)n);
    int jc = SLS_THREADS / n;
    while (jc > 1 && per_j * jc + 2 * n * sizeof(double) > SLS_ROW_LDS) --jc;
    *smem = per_j * jc;            // tube_row's region; callers add 2 n for the row results
    return jc;
}

// register length bucket of a row of Phi
static int nx_bucket(int nx) { return nx <= 8 ? 8 : (nx <= 16 ? 16 : 32); }

template <int MODE, int NXB>
__global__ void __launch_bounds__(SLS_THREADS) sls_tube_kernel(TubeRowArgs a, double* out_sig) {
    const int k = blockIdx.x, b = blockIdx.y;
    extern __shared__ double sm[];
    const int n = a.nx + a.nu;
    double* mo = sm;
    double* so = sm + n;
    tube_row<MODE, NXB>(a, row_ref(a, b, k), k, sm + 2 * n, mo, so);
    const size_t o = ((size_t)b * a.N + k) * n;
    for (int q = threadIdx.x; q < n; q += blockDim.x) {
        if (MODE == ROW_E) {
            out_sig[o + q] = so[q];
        } else {
            a.mu[o + q] = mo[q];
            a.sigma[o + q] = so[q];
        }
    }
}

typedef double sls_p2 __attribute__((ext_vector_type(2), aligned(8)));

// M[row][col] of a matrix with rows of C elements, 0 outside (a row past its end is
// out of the descriptor's range)
__device__ __forceinline__ double element_at(__amdgpu_buffer_rsrc_t M, int C, int row, int col) {
    union { sls_u2 u; double d; } x;
    x.u = __builtin_amdgcn_raw_buffer_load_b64(M, 8 * (row * C + col), 0, 0);
    return col < C ? x.d : 0.0;
}

// The disturbance part sum_j |Phi_{k,j} E_j| 1 of tube row k on FP64 MFMA for n > 8
// rows (RT = ceil(n / 16), CT = ceil(nw / 16) tiles): one workgroup per
// (trajectory, k), wave w takes the blocks j = w, w + 4, ...  A block is one
// zero-padded product (A fragments from Phi_{k,j}, B fragments from E_j, both
// straight from memory); the absolute values of its entries are added up over
// j.  The rounding allowance needs |Phi| |E| 1 = |Phi| (|E| 1): the row sums of
// |E_j| come from the B fragments by additions within 16 lanes, and the product with
// them runs on the VALU beside the MFMAs.
//
// What bounds it: the padded products (72 MFMA a block at nx = 30: 94 us for 64 x 40
// steps) with the address and masking work beside them, and reading Phi (479 MB
// there: 98 us).  The fragments of the next group of states are read during this
// group's products.  64 x 40 at nx = 30: 0.27 ms (VALU rows: 1.24 ms), at nx = 18
// 0.09 ms (0.305 ms); 256 x 40 at nx = 12: 0.097 ms (3 us more with |Phi| |E| as a
// second MFMA product).  Several rows k a workgroup, to share E_j, was slower
// (0.28 and 0.33 ms with two and four rows at nx = 30).
template <int RT, int CT>
__global__ void __launch_bounds__(256) sls_tube_e_mfma_kernel(TubeRowArgs a, double* out_sig) {
    const int k = blockIdx.x, b = blockIdx.y;
    const int nx = a.nx, nw = a.nw, N = a.N, n = nx + a.nu;
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    __shared__ double redT[4][16 * RT];
    __shared__ double redG[4][4][16 * RT];
    const double* prow = a.phi + (((size_t)b * N + k) * N) * n * nx;
    const double* Eb = a.E + (size_t)b * N * nx * nw;
    const int nch = (nx + 15) >> 4;              // groups of 16 states (four k-steps)
    const int nit = wave < k ? ((k - 1 - wave) / 4 + 1) * nch : 0;
    // a group's fragments: k-step t of lane group lq takes state l = 16 g + 4 lq + t, so a
    // lane's four entries of a Phi row are one 32-byte piece of a 128-byte line
    auto fetch = [&](int it, double (&A)[RT][4], double (&B)[4][CT]) {
        const int q = it / nch, j = wave + 4 * q, l0 = 16 * (it - q * nch) + 4 * lq;
        const auto rP = matrix_rsrc(prow + (size_t)j * n * nx, n * nx), rE = matrix_rsrc(Eb + (size_t)j * nx * nw, nx * nw);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                union { sls_u4 u; double d[2]; } x;
                x.u = __builtin_amdgcn_raw_buffer_load_b128(rP, 8 * ((16 * r + lr) * nx + l0 + 2 * h), 0, 0);
                A[r][2 * h] = l0 + 2 * h < nx ? x.d[0] : 0.0;
                A[r][2 * h + 1] = l0 + 2 * h + 1 < nx ? x.d[1] : 0.0;
            }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c) B[t][c] = element_at(rE, nw, l0 + t, 16 * c + lr);
    };
    sls_d4 T[RT], D[RT][CT];
    double G[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        T[r] = sls_d4{0.0, 0.0, 0.0, 0.0};
        G[r] = 0.0;
#pragma unroll
        for (int c = 0; c < CT; ++c) D[r][c] = sls_d4{0.0, 0.0, 0.0, 0.0};
    }
    double av[RT][4], bv[4][CT], an[RT][4], bn[4][CT];
    auto multiply = [&](int it) {
        const int c0 = it % nch, left = nx - 16 * c0;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (t >= left) break;
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    D[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[r][t], bv[t][c], D[r][c], 0, 0, 0);
            double e1 = 0.0;
#pragma unroll
            for (int c = 0; c < CT; ++c) e1 += fabs(bv[t][c]);
            e1 = sum16(e1);
#pragma unroll
            for (int r = 0; r < RT; ++r) G[r] = fma(fabs(av[r][t]), e1, G[r]);
        }
        if (c0 == nch - 1) {                     // block j complete
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int c = 0; c < CT; ++c) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) T[r][i] += fabs(D[r][c][i]);
                    D[r][c] = sls_d4{0.0, 0.0, 0.0, 0.0};
                }
        }
    };
    if (nit > 0) fetch(0, an, bn);
    for (int it = 0; it < nit; ++it) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
#pragma unroll
            for (int r = 0; r < RT; ++r) av[r][t] = an[r][t];
#pragma unroll
            for (int c = 0; c < CT; ++c) bv[t][c] = bn[t][c];
        }
        if (it + 1 < nit) fetch(it + 1, an, bn);
        multiply(it);
    }
    // the sixteen columns of each row (row 16 r + 4 i + lq), then the waves
#pragma unroll
    for (int r = 0; r < RT; ++r) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double t = sum16(T[r][i]);
            if (lr == 0) redT[wave][16 * r + 4 * i + lq] = t;
        }
        redG[wave][lq][16 * r + lr] = G[r];
    }
    __syncthreads();
    if (tid < n) {
        double sv = 0.0, g = 0.0;
        for (int w = 0; w < 4; ++w) {
            sv += redT[w][tid];
            for (int q = 0; q < 4; ++q) g += redG[w][q][tid];
        }
        // depth of the sums: nx products per entry inside the MFMA, k blocks, 4 waves, 16 columns
        const double coef = (double)(nx + k * (nw + 1) + 64) * 0x1p-52;
        sv = sv + coef * g * (1.0 + 0x1p-50) + 0x1p-1000;
        if (!isfinite(g) || !isfinite(sv)) sv = INFINITY;
        if (k == 0) sv = 0.0;
        out_sig[((size_t)b * N + k) * n + tid] = sv;
    }
}

template <int RT>
static void launch_tube_e_mfma(const TubeRowArgs& a, int batch, double* out_sig, hipStream_t s) {
    const dim3 grid((unsigned)a.N, (unsigned)batch);
    switch ((a.nw + 15) / 16) {
    case 1: hipLaunchKernelGGL((sls_tube_e_mfma_kernel<RT, 1>), grid, dim3(256), 0, s, a, out_sig); break;
    case 2: hipLaunchKernelGGL((sls_tube_e_mfma_kernel<RT, 2>), grid, dim3(256), 0, s, a, out_sig); break;
    case 3: hipLaunchKernelGGL((sls_tube_e_mfma_kernel<RT, 3>), grid, dim3(256), 0, s, a, out_sig); break;
    default: hipLaunchKernelGGL((sls_tube_e_mfma_kernel<RT, 4>), grid, dim3(256), 0, s, a, out_sig); break;
    }
}

// The same for one small size (n = NX + NU = 8 rows, nw <= 8) on the VALU: a lane
// holds row i of tube row k (eight rows, eight k a wave, five waves: 40 k a
// workgroup) and the wave walks j in step, so that E_j and |E_j| 1 are broadcasts
// from LDS and every lane's row of Phi_{k,j} is one 48-byte read, four j ahead.
//
// What bounds it: reading Phi (77 MB at 256 x 40: 16 us) and one wave's walk over
// up to 39 blocks.  256 x 40: 0.036 ms (a workgroup per row k, two barriers a chunk
// and the sums over its slots through LDS: 0.047 ms); 1,024 x 40: 0.108 ms (0.173 ms).
// At other horizons, the whole fixed point with it and with a workgroup per row: 256 x 10
// 41 and 41, 256 x 20 69 and 71, 256 x 80 305 and 341, 1,024 x 20 136 and 162 us; few long
// trajectories leave it too few waves: 64 x 150 699 and 663, 16 x 300 2,107 and 1,942.
template <int NX, int NU>
__global__ void __launch_bounds__(320) sls_tube_e_lane_kernel(TubeRowArgs a, double* out_sig) {
    constexpr int n = NX + NU, NW = 8, KW = 40, CH = 40, JU = 4;   // k a workgroup, staged j, j read ahead
    static_assert(n == 8 && NX % 2 == 0, "eight lanes per tube row");
    const int b = blockIdx.y, N = a.N, nw = a.nw;
    __shared__ double sE[CH][NX][NW];
    __shared__ double se[CH][NX];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = KW * blockIdx.x + 8 * wave;               // first k of this wave
    const int k = kw + (lane >> 3), i = lane & 7, kc = min(k, N - 1);
    const int kend = min(kw + 7, N - 1);                     // blocks j < kend matter to the wave
    const int kblk = min(KW * (int)blockIdx.x + KW - 1, N - 1);
    const double* row = a.phi + ((((size_t)b * N + kc) * N) * n + i) * NX;
    const double* Eb = a.E + (size_t)b * N * NX * nw;
    double s = 0.0, g = 0.0;
    sls_p2 rn[JU][NX / 2];
    auto fetch = [&](int u, int j) {                         // entries j >= k are read but not used
#pragma unroll
        for (int q = 0; q < NX / 2; ++q)
            rn[u][q] = *reinterpret_cast<const sls_p2*>(row + (size_t)min(j, N - 1) * n * NX + 2 * q);
    };
    for (int c0 = 0; c0 < kblk; c0 += CH) {
        const int cnt = min(CH, kblk - c0);
        __syncthreads();
        for (int q = tid; q < cnt * NX * NW; q += 320) {
            const int jl = q / (NX * NW), l = (q / NW) % NX, w = q % NW;
            sE[jl][l][w] = w < nw ? Eb[((size_t)(c0 + jl) * NX + l) * nw + w] : 0.0;
        }
        __syncthreads();
        for (int q = tid; q < cnt * NX; q += 320) {
            const int jl = q / NX, l = q % NX;
            double t = 0.0;
            for (int w = 0; w < NW; ++w) t += fabs(sE[jl][l][w]);
            se[jl][l] = t;
        }
        __syncthreads();
        const int je = min(c0 + cnt, kend);
#pragma unroll
        for (int u = 0; u < JU; ++u) fetch(u, c0 + u);
        for (int j = c0; j < je; j += JU) {
#pragma unroll
            for (int u = 0; u < JU; ++u) {
                double r[NX];
#pragma unroll
                for (int q = 0; q < NX / 2; ++q) { r[2 * q] = rn[u][q][0]; r[2 * q + 1] = rn[u][q][1]; }
                fetch(u, j + u + JU);
                const int jl = min(j + u, je - 1) - c0;
                double t[NW], gg = 0.0, ss = 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) t[w] = 0.0;
#pragma unroll
                for (int l = 0; l < NX; ++l) {
                    gg = fma(fabs(r[l]), se[jl][l], gg);
#pragma unroll
                    for (int w = 0; w < NW; ++w) t[w] = fma(r[l], sE[jl][l][w], t[w]);
                }
#pragma unroll
                for (int w = 0; w < NW; ++w) ss += fabs(t[w]);
                if (j + u < k && j + u < je) { s += ss; g += gg; }
            }
        }
    }
    if (k < N) {
        // depth of the sums: NX products, NW columns, k blocks
        const double coef = (double)(NX + k * (nw + 1) + 64) * 0x1p-52;
        s = s + coef * g * (1.0 + 0x1p-50) + 0x1p-1000;
        if (!isfinite(g) || !isfinite(s)) s = INFINITY;
        if (k == 0) s = 0.0;
        out_sig[((size_t)b * N + k) * n + i] = s;
    }
}

template <int MODE>
static void launch_tube(const TubeRowArgs& a, int batch, double* out_sig, hipStream_t s) {
    size_t smem;
    TubeRowArgs t = a;
    t.jc = tube_jc(a.nx, a.nu, a.nw, MODE, &smem);
    smem += 2 * (a.nx + a.nu) * sizeof(double);
    const dim3 grid((unsigned)a.N, (unsigned)batch);
    switch (nx_bucket(a.nx)) {
    case 8: hipLaunchKernelGGL((sls_tube_kernel<MODE, 8>), grid, dim3(SLS_THREADS), smem, s, t, out_sig); break;
    case 16: hipLaunchKernelGGL((sls_tube_kernel<MODE, 16>), grid, dim3(SLS_THREADS), smem, s, t, out_sig); break;
    default: hipLaunchKernelGGL((sls_tube_kernel<MODE, 32>), grid, dim3(SLS_THREADS), smem, s, t, out_sig); break;
    }
}

// ------------------------------------------------------------ disturbance error

// FP64 interval sine and cosine of [lo, hi] from the library values at its ends
// (sa, sb = sin lo, sin hi; ca, cb = cos lo, cos hi): widened by 2^-40 relative
// plus 2^-100 absolute, +-1 where a critical point may lie inside (tested
// against an outward pi) and everywhere for wide or far-out intervals, whose library
// values are not needed (far out they cost several times as much).
constexpr double SLS_PI_LO = 3.141592653589793115997963468544185161590576171875;

__device__ __forceinline__ bool sls_wide(double lo, double hi) {
    return !(hi - lo < 2.0 * SLS_PI_LO) || fabs(lo) > 1024.0 || fabs(hi) > 1024.0;
}

__device__ void sls_sincos(double lo, double hi, double sa, double sb, double ca, double cb, double* sl, double* sh,
                           double* cl, double* ch) {
    const double PI_LO = SLS_PI_LO;
    const double PI_HI = 3.141592653589793560087173318606801331043243408203125;
    if (sls_wide(lo, hi)) {
        *sl = -1.0; *sh = 1.0; *cl = -1.0; *ch = 1.0;
        return;
    }
    auto wdn = [](double x) { return x - fabs(x) * 0x1p-40 - 0x1p-100; };
    auto wup = [](double x) { return x + fabs(x) * 0x1p-40 + 0x1p-100; };
    double s0 = wdn(fmin(sa, sb)), s1 = wup(fmax(sa, sb));
    double c0 = wdn(fmin(ca, cb)), c1 = wup(fmax(ca, cb));
    auto may = [&](double frac) {
        const double x0 = frac * PI_LO;
        const double m = ceil((lo - x0) / (2.0 * PI_HI) - 1e-12);
        const double crit = x0 + m * 2.0 * (m >= 0 ? PI_LO : PI_HI);
        return crit <= hi + 1e-12;
    };
    if (may(0.5)) s1 = 1.0;
    if (may(-0.5)) s0 = -1.0;
    if (may(0.0)) c1 = 1.0;
    if (may(1.0)) c0 = -1.0;
    *sl = fmax(s0, -1.0); *sh = fmin(s1, 1.0);
    *cl = fmax(c0, -1.0); *ch = fmin(c1, 1.0);
}

__device__ __forceinline__ double rdn(double x) { return x - fabs(x) * 0x1p-52 - 0x1p-1000; }
__device__ __forceinline__ double rup(double x) { return x + fabs(x) * 0x1p-52 + 0x1p-1000; }

// ends of theta's interval over the tube set
__device__ __forceinline__ void thrust_theta(double zt, double mut, double sgt, double* lo, double* hi) {
    *lo = rdn(zt + mut - sgt);
    *hi = rup(zt + mut + sgt);
}

// half-width of a thrust column's disturbance error on a node's vx (comp 3) or vz
// (comp 4) row, from theta's interval and the library values at its ends
__device__ double thrust_rdist(int comp, double lo, double hi, double sa, double sb, double ca, double cb, double e0,
                               double c) {
    if (!(lo <= hi) || !isfinite(lo) || !isfinite(hi)) return INFINITY;
    double sl, sh, cl, ch;
    sls_sincos(lo, hi, sa, sb, ca, cb, &sl, &sh, &cl, &ch);
    // vx: -c [sin], vz: c [cos]; products of the point c >= 0 rounded outward
    const double a = comp == 3 ? rdn(-c * sh) : rdn(c * cl);
    const double bq = comp == 3 ? rup(-c * sl) : rup(c * ch);
    return rup(fmax(fabs(rup(bq - e0)), fabs(rdn(a - e0))));
}

// the same for any row l (0 off the (vx, vz) rows), from the tube's theta entries
__device__ double thrust_rdist_row(int l, double zt, double mut, double sgt, double e0, double c) {
    const int comp = l % 6;
    if (comp != 3 && comp != 4) return 0.0;
    double lo, hi;
    thrust_theta(zt, mut, sgt, &lo, &hi);
    double sa = 0.0, sb = 0.0, ca = 0.0, cb = 0.0;
    if (!sls_wide(lo, hi)) {
        sincos(lo, &sa, &ca);
        sincos(hi, &sb, &cb);
    }
    return thrust_rdist(comp, lo, hi, sa, sb, ca, cb, e0, c);
}

struct EDiag { double e[SLS_MAX_NX]; };

// E(z_k) = [diag(e) | thrust columns], [units][nx][nx + U]
__global__ void sls_disturbance_kernel(const double* z, EDiag e, double c, int nx, int U, int64_t units,
                                       double* E) {
    const int nw = nx + U;
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= units * nx * nw) return;
    const int64_t u = q / ((int64_t)nx * nw);
    const int r = (int)((q / nw) % nx), w = (int)(q % nw);
    double val = 0.0;
    if (w < nx) val = w == r ? e.e[r] : 0.0;
    else {
        const int i = w - nx;
        const double th = z[u * nx + 6 * i + 2];
        if (r == 6 * i + 3) val = -c * sin(th);
        else if (r == 6 * i + 4) val = c * cos(th);
    }
    E[q] = val;
}

// ------------------------------------------------------------ fixed point

struct FpRowArgs {
    TubeRowArgs t;           // cbar, rbar: workspace (written here through cbar_w, rbar_w)
    double* cbar_w; double* rbar_w;
    const double* z; const double* v;
    const double* rlo_s; const double* rhi_s;   // [b][nx] bound of step k-1 (staging)
    double* zs; double* vs; double* mus; double* sgs;   // staging for the bound of step k
    double* r_lo; double* r_hi;                  // [b][N][nx] outputs (may be NULL)
    uint32_t* certified;                         // [b] (may be NULL)
    double thrust_c;                             // thrust dt / m (0: constant E)
    double pad;
    int U;
};

// Row launch of step k (k = N: only finishes step N-1).  One workgroup per trajectory.
template <int NXB>
__global__ void __launch_bounds__(SLS_THREADS) sls_fp_row_kernel(FpRowArgs a, int k) {
    const int b = blockIdx.x;
    const TubeRowArgs& t = a.t;
    const int nx = t.nx, nu = t.nu, n = nx + nu, N = t.N, nw = t.nw;
    extern __shared__ double sm[];
    double* mo = sm;
    double* so = sm + n;
    const int tid = threadIdx.x;
    if (k > 0) {
        // residual zonotope of step k-1: bound + disturbance error, outward
        const int kp = k - 1;
        for (int l = tid; l < nx; l += blockDim.x) {
            double lo = a.rlo_s[(size_t)b * nx + l], hi = a.rhi_s[(size_t)b * nx + l];
            if (a.thrust_c > 0.0) {
                const int node = l / 6, th = 6 * node + 2;
                const size_t ob = ((size_t)b * N + kp);
                const double e0 = t.E[(ob * nx + l) * nw + (nw - a.U + node)];
                const double s = thrust_rdist_row(l, a.z[ob * nx + th], t.mu[ob * n + th], t.sigma[ob * n + th], e0,
                                                  a.thrust_c);
                if (s != 0.0) {
                    lo = rdn(lo - s);
                    hi = rup(hi + s);
                }
            }
            const size_t o = ((size_t)b * N + kp) * nx + l;
            if (a.r_lo) { a.r_lo[o] = lo; a.r_hi[o] = hi; }
            double cb = 0.5 * (lo + hi), rb = fmax(hi - cb, cb - lo);
            rb = rup(rup(rb) + a.pad);
            if (!isfinite(lo) || !isfinite(hi)) { cb = NAN; rb = INFINITY; }
            a.cbar_w[o] = cb;
            a.rbar_w[o] = rb;
        }
        __syncthreads();
    }
    if (k == N) {
        if (a.certified && tid == 0) {
            // every tube entry and residual finite: the causal pass reached C = F(C)
            bool fin = true;
            for (int q = 0; q < N * n && fin; ++q) fin = isfinite(t.sigma[(size_t)b * N * n + q]);
            for (int q = 0; q < N * nx && fin; ++q) fin = isfinite(t.rbar[(size_t)b * N * nx + q]);
            a.certified[b] = fin ? 1u : 0u;
        }
        return;
    }
    tube_row<ROW_NOE, NXB>(t, row_ref(t, b, k), k, sm + 2 * n, mo, so);
    const size_t o = ((size_t)b * N + k) * n;
    for (int q = tid; q < n; q += blockDim.x) {
        t.mu[o + q] = mo[q];
        t.sigma[o + q] = so[q];
        a.mus[(size_t)b * n + q] = mo[q];
        a.sgs[(size_t)b * n + q] = so[q];
    }
    const size_t ob = (size_t)b * N + k;
    for (int q = tid; q < nx; q += blockDim.x) a.zs[(size_t)b * nx + q] = a.z[ob * nx + q];
    for (int q = tid; q < nu; q += blockDim.x) a.vs[(size_t)b * nu + q] = a.v[ob * nu + q];
}

// Chain dynamics: the whole causal pass of one trajectory in one workgroup, its
// nominal, disturbance parts, thrust entries and residual zonotopes in LDS.
// The tube row k + 1 needs the residual of step k only through its last block
// Phi_{k+1,k}, so the waves take different parts of step k:
//   A  others  row k = the sums over j < k - 1 (formed during step k - 1) plus the
//              block Phi_{k,k-1} (in LDS) times the residual of step k - 1
//   B  wave 0  the path-based bound of the unit (z_k, v_k) + mu_k +- sigma_k (U lanes)
//      wave 1  the thrust disturbance error over theta's interval (two lanes a node,
//              one library call each)
//      others  the sums of row k + 1 over j < k: thread p holds the two entries
//              2p, 2p + 1 of every block, so a block is one coalesced read; the first
//              SLS_FP_PF blocks were read during step k - 1
//   C  wave 0  the residual zonotope of step k;  others: the partial sums of B
//              added up per row, the block Phi_{k+1,k} to LDS
// with one LDS barrier after each.
//
// FOLD: the stream's places are dealt to two waves, each thread takes several one after the
// other (the same sums in the same order, bit for bit) and nothing is read ahead.  With its
// 160 VGPRs a compute unit holds twelve waves: three workgroups of four instead of one of
// seven (nx = 12) or eight, or two of six.
//
// What bounds it: 40 dependent steps, each the latency of A, of the slowest of B
// (the bound at small nx, the stream of the row at nx = 30: up to 374 KB a step for
// one compute unit) and of C.  256 x 40 steps at nx = 6: 0.092 ms (rows, bound and
// disturbance error one after the other: 0.224 ms); at nx = 12 0.195 ms (0.378 ms);
// 64 x 40 at nx = 30 0.300 ms (1.33 ms).
constexpr int SLS_FP_PF = 8;             // blocks of the next row read one step ahead
constexpr int SLS_FP_MAX_THREADS = 768, SLS_FOLD_THREADS = 256;

struct FpChainArgs {
    const double* phi; const double* E; const double* sigE;
    const double* z; const double* v;
    double* mu; double* sigma; double* r_lo; double* r_hi;
    uint32_t* certified;
    double thrust_c;
    int nu, nw, N;
    int npos, slots;         // two-entry positions of a block; blocks in flight across the stream waves
    // node-pass constants
    int U;
    double c, kL, L0, pad;
    int compact;
};

template <bool FOLD>
__global__ void __launch_bounds__(SLS_FP_MAX_THREADS) sls_fp_chain_kernel(FpChainArgs a) {
    const int b = blockIdx.x;
    const int U = a.U, nx = 6 * U, nu = a.nu, n = nx + nu, N = a.N, nw = a.nw;
    extern __shared__ double sm[];
    const int nst = a.npos * a.slots;            // places in the row stream
    double* mo = sm;                    // n
    double* so = mo + n;                // n
    double* rl = so + n;                // nx
    double* rh = rl + nx;               // nx
    double* rd = rh + nx;               // nx     disturbance error of step k
    double* base = rd + nx;             // 3*n    sums of the next row over the earlier steps
    double* zl = base + 3 * n;          // N*nx
    double* vl = zl + (size_t)N * nx;   // N*nu
    double* sel = vl + (size_t)N * nu;  // N*n
    double* eth = sel + (size_t)N * n;  // N*2*U  E_k entries of the thrust columns (vx, vz rows)
    double* cbl = eth + (size_t)N * 2 * U;      // N*nx
    double* rbl = cbl + (size_t)N * nx;         // N*nx
    double* blk = rbl + (size_t)N * nx;         // n*nx   Phi_{k,k-1}
    double* part = blk + n * nx;                // 3*nst
    SpringOut* s_sp = reinterpret_cast<SpringOut*>(part + 3 * nst);             // [U]
    uint32_t* s_flag = reinterpret_cast<uint32_t*>(s_sp + U);                   // [2]: flags, all finite
    const int tid = threadIdx.x, bs = blockDim.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t b0 = (size_t)b * N;
    const double* phib = a.phi + b0 * N * n * nx;
    for (int q = tid; q < N * nx; q += bs) zl[q] = a.z[b0 * nx + q];
    for (int q = tid; q < N * nu; q += bs) vl[q] = a.v[b0 * nu + q];
    for (int q = tid; q < N * n; q += bs) sel[q] = a.sigE[b0 * n + q];
    for (int q = tid; q < N * 2 * U; q += bs) {
        const int k = q / (2 * U), u = (q >> 1) % U, e = q & 1;
        eth[q] = a.thrust_c > 0.0 ? a.E[((b0 + k) * nx + 6 * u + 3 + e) * nw + (nw - U + u)] : 0.0;
    }
    for (int q = tid; q < nx; q += bs) rd[q] = 0.0;
    if (tid == 0) s_flag[1] = 1u;
    __syncthreads();
    // one loop a role, with the same three barriers in each (the role is uniform over a
    // wave), so that a wave holds the registers of its own part only
    if (wave == 0) {
        const int lt = lane / U, i = lane - lt * U;
        for (int k = 0; k < N; ++k) {
            lds_barrier();                       // A done: row k in mo, so
            if (lane == 0) s_flag[0] = 0u;
            const TileRef t0{zl + (size_t)k * nx, vl + (size_t)k * nu, mo, so, rl, rh, nullptr, nullptr, nullptr, 1};
            NodeIn d;
            node_load(t0, U, lt, i, d);
            wave_lds_fence();                    // s_flag cleared
            node_pass<true>(a, t0, d, lt, i, s_sp, s_flag);
            lds_barrier();                       // B done
            if (lane < nx) {
                const int l = lane;
                double lo = rl[l], hi = rh[l];
                const double s = rd[l];
                if (s != 0.0) {
                    lo = rdn(lo - s);
                    hi = rup(hi + s);
                }
                double c = 0.5 * (lo + hi), r = fmax(hi - c, c - lo);
                r = rup(rup(r) + a.pad);
                if (!isfinite(lo) || !isfinite(hi)) { c = NAN; r = INFINITY; }
                cbl[(size_t)k * nx + l] = c;
                rbl[(size_t)k * nx + l] = r;
                if (!isfinite(r)) s_flag[1] = 0u;
                if (a.r_lo) { a.r_lo[(b0 + k) * nx + l] = lo; a.r_hi[(b0 + k) * nx + l] = hi; }
            }
            lds_barrier();                       // C done
        }
    } else if (wave == 1) {
        const int u = lane >> 1, e = lane & 1, th = 6 * u + 2;
        const bool mine = a.thrust_c > 0.0 && lane < 2 * U;
        for (int k = 0; k < N; ++k) {
            lds_barrier();
            if (mine) {
                double lo, hi, sx = 0.0, cx = 0.0;
                thrust_theta(zl[(size_t)k * nx + th], mo[th], so[th], &lo, &hi);
                if (!sls_wide(lo, hi)) sincos(e ? hi : lo, &sx, &cx);
                const double sy = __shfl_xor(sx, 1), cy = __shfl_xor(cx, 1);
                rd[6 * u + 3 + e] = thrust_rdist(3 + e, lo, hi, e ? sy : sx, e ? sx : sy, e ? cy : cx, e ? cx : cy,
                                                 eth[((size_t)k * U + u) * 2 + e], a.thrust_c);
            }
            lds_barrier();
            lds_barrier();
        }
    } else {
        // this thread's place in the row stream (FOLD: its first one)
        const int st = tid - 128, lanes = bs - 128, hx = nx >> 1, per = hx * a.slots;
        const bool streams = st < nst;
        int pos, slot, l2, mine;
        auto place = [&](int q) {
            pos = q % a.npos;
            slot = q / a.npos;
            l2 = 2 * (pos % hx);
            mine = (pos / hx) * per + slot * hx + pos % hx;                      // partial sums, row by row
        };
        place(streams ? st : 0);
        auto load = [&](int k, int j) {          // entries 2 pos, 2 pos + 1 of Phi_{k,j}
            return *reinterpret_cast<const sls_p2*>(phib + ((size_t)k * N + j) * n * nx + 2 * pos);
        };
        sls_p2 pf[SLS_FP_PF], nb = {0.0, 0.0};
#pragma unroll
        for (int q = 0; q < SLS_FP_PF; ++q) pf[q] = sls_p2{0.0, 0.0};
        for (int k = 0; k < N; ++k) {
            // A: row k (four lanes a row)
            auto row_k = [&](int w) {
                const int i = w >> 2, q = w & 3;
                double m = 0.0, s = 0.0, g = 0.0;
                if (k > 0) {
                    const double* cb = cbl + (size_t)(k - 1) * nx;
                    const double* rb = rbl + (size_t)(k - 1) * nx;
                    for (int l = q; l < nx; l += 4) {
                        const double r = blk[i * nx + l], ap = fabs(r), c = cb[l], h = rb[l];
                        m = fma(r, c, m);
                        s = fma(ap, h, s);
                        g = fma(ap, fabs(c) + h, g);
                    }
                }
                m = sum4(m);
                s = sum4(s);
                g = sum4(g);
                if (q == 0) {
                    if (k > 1) { m += base[i]; s += base[n + i]; g += base[2 * n + i]; }
                    // rounding of the sums: at most 2 k + nx + 72 additions deep (two entries a
                    // block in the stream, one block a slot at least), each within 2^-53 of the
                    // magnitudes g; doubled for the centre's error and the final additions
                    const double coef = (double)(nx + k * max(nw + 1, 2) + 72) * 0x1p-52;
                    s = s + coef * g * (1.0 + 0x1p-50) + 0x1p-1000;
                    const double se = sel[(size_t)k * n + i];
                    s = s + se;
                    s = s + fabs(s) * 0x1p-52;
                    if (!isfinite(g) || !isfinite(s) || !isfinite(se)) { m = 0.0; s = INFINITY; }
                    if (k == 0) { m = 0.0; s = 0.0; }
                    mo[i] = m;
                    so[i] = s;
                    a.mu[(b0 + k) * n + i] = m;
                    a.sigma[(b0 + k) * n + i] = s;
                    if (!isfinite(s)) s_flag[1] = 0u;
                }
            };
            if constexpr (FOLD) {
                for (int w = st; w < 4 * n; w += lanes) row_k(w);
            } else if (st < 4 * n) {
                row_k(st);
            }
            lds_barrier();
            // B: the next row over the residuals known before this step
            if (streams && k + 1 < N) {
                double m, s, g;
                auto add = [&](int j, sls_p2 r) {
                    const double* cb = cbl + (size_t)j * nx + l2;
                    const double* rb = rbl + (size_t)j * nx + l2;
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const double ap = fabs(r[e]);
                        m = fma(r[e], cb[e], m);
                        s = fma(ap, rb[e], s);
                        g = fma(ap, fabs(cb[e]) + rb[e], g);
                    }
                };
                auto rest = [&](int j) {         // blocks j, j + slots, ... below k
                    for (; j < k; j += SLS_FP_PF * a.slots) {
                        sls_p2 r[SLS_FP_PF];
#pragma unroll
                        for (int q = 0; q < SLS_FP_PF; ++q) r[q] = load(k + 1, min(j + q * a.slots, k - 1));
#pragma unroll
                        for (int q = 0; q < SLS_FP_PF; ++q)
                            if (j + q * a.slots < k) add(j + q * a.slots, r[q]);
                    }
                };
                auto put = [&]() {
                    part[mine] = m;
                    part[nst + mine] = s;
                    part[2 * nst + mine] = g;
                };
                if constexpr (FOLD) {
                    for (int q = st; q < nst; q += lanes) {
                        place(q);
                        if (slot == 0) nb = load(k + 1, k);
                        m = s = g = 0.0;
                        rest(slot);
                        put();
                        if (slot == 0) { blk[2 * pos] = nb[0]; blk[2 * pos + 1] = nb[1]; }   // (A has read the last one)
                    }
                } else {
                    if (slot == 0) nb = load(k + 1, k);
                    m = s = g = 0.0;
                    int j = slot;
#pragma unroll
                    for (int q = 0; q < SLS_FP_PF; ++q, j += a.slots)
                        if (j < k) add(j, pf[q]);
                    rest(j);
                    if (k + 2 < N) {
#pragma unroll
                        for (int q = 0; q < SLS_FP_PF; ++q) pf[q] = load(k + 2, min(slot + q * a.slots, k));
                    }
                    put();
                }
            }
            lds_barrier();
            // C: eight lanes a row over its nx / 2 positions in every slot
            if (k + 1 < N) {
                auto row_sums = [&](int w) {
                    const int i = w >> 3;
                    double m = 0.0, s = 0.0, g = 0.0;
                    for (int q = i * per + (w & 7); q < (i + 1) * per; q += 8) {
                        m += part[q];
                        s += part[nst + q];
                        g += part[2 * nst + q];
                    }
                    m = sum8(m);
                    s = sum8(s);
                    g = sum8(g);
                    if ((w & 7) == 0) { base[i] = m; base[n + i] = s; base[2 * n + i] = g; }
                };
                if constexpr (FOLD) {
                    for (int w = st; w < 8 * n; w += lanes) row_sums(w);
                } else if (st < 8 * n) {
                    row_sums(st);
                }
                if (!FOLD && streams && slot == 0) { blk[2 * pos] = nb[0]; blk[2 * pos + 1] = nb[1]; }
            }
            lds_barrier();
        }
    }
    __syncthreads();
    if (a.certified && tid == 0) a.certified[b] = s_flag[1];
}

// Slots and LDS bytes of sls_fp_chain_kernel; 0: too large for the one-launch form.
// Slots: blocks side by side in the row stream.  At nx = 6 (24 positions a block) two
// stream waves hold five, so that the blocks read ahead cover 40 steps and two
// workgroups share a compute unit (256 / 1,024 trajectories of 40 steps: 95 / 194 us;
// with five stream waves 101 / 396 us); at 20 steps the number does not matter (256: 61
// us, with five waves 64), beyond the steps read ahead five waves are faster for few
// trajectories (256 x 80 270 and 248, 64 x 150 605 and 436 us).  Larger blocks need the five waves to keep a
// row's reads in flight (nx = 12: 197 us, with two waves 226 us); at least one slot.
// Fold: batches of more than a workgroup a compute unit, while a step's stream is short
// enough for two waves (positions of a block times N; the longer, the more the reads ahead
// matter).  No disturbance, us, unfolded and folded, in brackets a workgroup that took its
// phases one after the other:
//   nx = 12   512 x 40   552  498 (527)      nx = 18   2,048 x 25   1,763  1,478 (1,789)
//             512 x 64 1,124 1,173 (1,160)             8,192 x 10   2,082  1,216 (1,516)
//           2,048 x 40 2,162 1,668 (1,794)             1,024 x 40   2,061  2,037 (2,338)
//           2,048 x 64 4,439 4,067 (4,110)   nx = 24   8,192 x 10   2,544  1,864 (2,209)
//           8,192 x 10 1,747   863 (1,051)             2,048 x 30   3,394  3,369 (-)
//             512 x 80 1,454 1,591 (1,548)   nx = 30   8,192 x 10   3,511  3,235 (3,983)
static size_t fp_chain_plan(int nx, int nu, int U, int N, int batch, int* npos, int* slots, int* threads, bool* fold) {
    const int n = nx + nu;
    *npos = n * nx / 2;
    *slots = max(1, (*npos <= 24 ? 128 : 320) / *npos);
    const int stream = max(*npos * *slots, 8 * n);
    *threads = 128 + 64 * ((stream + 63) / 64);
    if (*threads > SLS_FP_MAX_THREADS) return 0;
    *fold = batch > 256 && *npos * N <= (batch > 1024 ? 7680 : 5376) && *threads > SLS_FOLD_THREADS;
    if (*fold) *threads = SLS_FOLD_THREADS;
    const size_t bytes = sizeof(double) * ((size_t)5 * n + 3 * nx + (size_t)N * (3 * nx + nu + n + 2 * U) + n * nx +
                                           (size_t)3 * *npos * *slots) +
                         sizeof(SpringOut) * U + 2 * sizeof(uint32_t);
    return bytes <= SLS_LDS_MAX ? bytes : 0;
}

struct SlsWorkspace {
    std::mutex mu;
    double* buf = nullptr;
    size_t cap = 0;
    WsFence fence;
};
static SlsWorkspace g_sls;

static bool dims_ok(int nx, int nu) { return nx >= 1 && nx <= SLS_MAX_NX && nu >= 0 && nu <= SLS_MAX_NU; }

}  // namespace leb

using namespace leb;

static int sls_responses(int32_t nx, int32_t nu, int32_t batch, int32_t N, const double* A, const double* B,
                         const double* qx, const double* qu, double* K, double* phi, bool zero, void* stream) {
    if (!dims_ok(nx, nu) || nu < 1 || batch < 0 || N < 0) return LEB_EINVAL;
    if (batch > 65535 || N > 65535) return LEB_ENOTSUP;
    if ((int64_t)batch * N * N == 0) return LEB_OK;
    if (!A || !B || !qx || !qu || !K || !phi) return LEB_EINVAL;
    const void* ptrs[] = {A, B, qx, qu, K, phi};
    for (const void* p : ptrs)
        if (!aligned8(p)) return LEB_EINVAL;
    RiccatiArgs a;
    a.A = A; a.B = B; a.qx = qx; a.qu = qu; a.K = K; a.phi = phi;
    a.nx = nx; a.nu = nu; a.N = N; a.zero = zero ? 1 : 0;
    hipStream_t st = (hipStream_t)stream;
    // the planar quadrotor has a kernel with eight lanes a chain (whole calls, new buffers: 1 x 40
    // steps 59 us, 256 x 40 89, 1,024 x 40 354; on the tiles 86, 244 and 964); all else runs
    // on the matrix cores
    if (nx == 6 && nu == 2)
        hipLaunchKernelGGL((sls_riccati_lane_kernel<6, 2>), dim3((unsigned)((N + 7) / 8), (unsigned)batch), dim3(64),
                           0, st, a);
    else if (nx > 16)
        launch_riccati_tile<2>(a, batch, st);
    else
        launch_riccati_tile<1>(a, batch, st);
    return hipGetLastError() == hipSuccess ? LEB_OK : LEB_EDEVICE;
}

extern "C" int leb_sls_responses(int32_t nx, int32_t nu, int32_t batch, int32_t N, const double* A, const double* B,
                                 const double* qx, const double* qu, double* K, double* phi, void* stream) {
    return sls_responses(nx, nu, batch, N, A, B, qx, qu, K, phi, false, stream);
}

extern "C" int leb_sls_responses_full(int32_t nx, int32_t nu, int32_t batch, int32_t N, const double* A,
                                      const double* B, const double* qx, const double* qu, double* K, double* phi,
                                      void* stream) {
    return sls_responses(nx, nu, batch, N, A, B, qx, qu, K, phi, true, stream);
}

extern "C" int leb_sls_tube_map(int32_t nx, int32_t nu, int32_t nw, int32_t batch, int32_t N, const double* phi,
                                const double* E, const double* c_bar, const double* rho_bar, double* mu,
                                double* sigma, void* stream) {
    if (!dims_ok(nx, nu) || nw < 0 || nw > SLS_MAX_NW || batch < 0 || N < 0) return LEB_EINVAL;
    if (batch > 65535 || N > 65535) return LEB_ENOTSUP;
    if ((int64_t)batch * N == 0) return LEB_OK;
    if (!phi || (nw > 0 && !E) || !c_bar || !rho_bar || !mu || !sigma) return LEB_EINVAL;
    const void* ptrs[] = {phi, E, c_bar, rho_bar, mu, sigma};
    for (const void* p : ptrs)
        if (p && !aligned8(p)) return LEB_EINVAL;
    TubeRowArgs a;
    a.phi = phi; a.E = E; a.cbar = c_bar; a.rbar = rho_bar; a.mu = mu; a.sigma = sigma; a.sigE = nullptr;
    a.nx = nx; a.nu = nu; a.nw = nw; a.N = N;
    launch_tube<ROW_FULL>(a, batch, nullptr, (hipStream_t)stream);
    return hipGetLastError() == hipSuccess ? LEB_OK : LEB_EDEVICE;
}

extern "C" int leb_linearize(const leb_dynamics* dyn, int32_t batch, int32_t N, const double* z, const double* v,
                             const double* e, double thrust, double* A, double* B, double* E, void* stream) {
    int rc = check_dynamics(dyn);
    if (rc != LEB_OK) return rc;
    if (dyn->kind != LEB_DYN_PQUAD_CHAIN) return LEB_ENOTSUP;
    if (batch < 0 || N < 0 || !(thrust >= 0.0) || !isfinite(thrust)) return LEB_EINVAL;
    const int64_t units = (int64_t)batch * N;
    if (units == 0) return LEB_OK;
    if (!z || !v || !A || !B || (E && !e)) return LEB_EINVAL;
    const void* ptrs[] = {z, v, A, B, E};
    for (const void* p : ptrs)
        if (p && !aligned8(p)) return LEB_EINVAL;
    const int nx = dyn->nx, U = dyn->n_units;
    if (units * nx * (nx + dyn->nu + nx + U) > ((int64_t)1 << 46)) return LEB_EINVAL;
    EDiag ed;
    if (E) {
        if (nx > SLS_MAX_NX) return LEB_ENOTSUP;
        for (int i = 0; i < nx; ++i) {
            if (!(e[i] >= 0.0) || !isfinite(e[i])) return LEB_EINVAL;
            ed.e[i] = e[i];
        }
    }
    hipStream_t s = (hipStream_t)stream;
    if ((rc = launch_chain_jacobians(dyn, units, z, v, A, B, s))) return rc;
    if (!E) return LEB_OK;
    const int64_t cnt = units * nx * (nx + U);
    hipLaunchKernelGGL(sls_disturbance_kernel, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s, z, ed,
                       thrust * dyn->dt / dyn->m, nx, U, units, E);
    return hipGetLastError() == hipSuccess ? LEB_OK : LEB_EDEVICE;
}

extern "C" int leb_sls_fixed_point(const leb_dynamics* dyn, int32_t batch, int32_t N, const double* z,
                                   const double* v, const double* phi, int32_t nw, const double* E, double thrust,
                                   double pad, double* mu, double* sigma, double* r_lo, double* r_hi,
                                   uint32_t* certified, void* stream) {
    int rc = check_dynamics(dyn);
    if (rc != LEB_OK) return rc;
    const int nx = dyn->nx, nu = dyn->nu, n = nx + nu;
    if (!dims_ok(nx, nu) || nw < 0 || nw > SLS_MAX_NW || batch < 0 || N < 0) return LEB_EINVAL;
    if (!(pad >= 0.0) || !isfinite(pad) || !(thrust >= 0.0) || !isfinite(thrust)) return LEB_EINVAL;
    const bool chain = dyn->kind == LEB_DYN_PQUAD_CHAIN;
    if (dyn->kind == LEB_DYN_LINEAR || dyn->kind == LEB_DYN_QUADRATIC || dyn->kind == LEB_DYN_SINCOS)
        return LEB_ENOTSUP;
    if (thrust > 0.0 && (!chain || nw < dyn->n_units)) return LEB_EINVAL;
    if (batch > 65535) return LEB_ENOTSUP;
    if ((int64_t)batch * N == 0) return LEB_OK;
    if (!z || (nu > 0 && !v) || !phi || (nw > 0 && !E) || !mu || !sigma || (!r_lo != !r_hi)) return LEB_EINVAL;
    const void* ptrs[] = {z, v, phi, E, mu, sigma, r_lo, r_hi};
    for (const void* p : ptrs)
        if (p && !aligned8(p)) return LEB_EINVAL;
    if (certified && (reinterpret_cast<uintptr_t>(certified) & 3u)) return LEB_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    std::lock_guard<std::mutex> lock(g_sls.mu);
    // cbar, rbar [b][N][nx]; sigE [b][N][n]; staging zs [b][nx], vs [b][nu], mus, sgs [b][n], rlo_s, rhi_s [b][nx]
    const size_t need = (size_t)batch * (2 * (size_t)N * nx + (size_t)N * n + nx + nu + 2 * n + 2 * nx) + 1;
    if (need > g_sls.cap) {
        if (g_sls.buf) (void)hipFree(g_sls.buf);
        g_sls.buf = nullptr;
        g_sls.cap = 0;
        if (hipMalloc(&g_sls.buf, need * sizeof(double)) != hipSuccess) return LEB_ENOMEM;
        g_sls.cap = need;
    }
    if ((rc = g_sls.fence.enter(s))) return rc;
    WsFenceScope leave{g_sls.fence, s};
    double* p = g_sls.buf;
    auto take = [&](size_t cnt) { double* q = p; p += cnt; return q; };
    FpRowArgs a;
    a.t.phi = phi; a.t.E = E; a.t.mu = mu; a.t.sigma = sigma;
    a.cbar_w = take((size_t)batch * N * nx);
    a.rbar_w = take((size_t)batch * N * nx);
    a.t.cbar = a.cbar_w;
    a.t.rbar = a.rbar_w;
    a.t.nx = nx; a.t.nu = nu; a.t.nw = nw; a.t.N = N;
    // the disturbance part of every tube entry first: it does not depend on the bounds,
    // so it runs over all (trajectory, step) rows at once
    double* sigE = take((size_t)batch * N * n);
    a.t.sigE = sigE;
    if (nw > 0 && n > 32)
        launch_tube_e_mfma<3>(a.t, batch, sigE, s);
    else if (nw > 0 && n > 16)
        launch_tube_e_mfma<2>(a.t, batch, sigE, s);
    else if (nw > 0 && n > 8)
        launch_tube_e_mfma<1>(a.t, batch, sigE, s);
    else if (nx == 6 && nu == 2 && nw > 0 && nw <= 8)
        hipLaunchKernelGGL((sls_tube_e_lane_kernel<6, 2>), dim3((unsigned)((N + 39) / 40), (unsigned)batch), dim3(320), 0,
                           s, a.t, sigE);
    else
        launch_tube<ROW_E>(a.t, batch, sigE, s);
    size_t smem;
    a.t.jc = tube_jc(nx, nu, nw, ROW_NOE, &smem);
    smem += 2 * n * sizeof(double);
    const int nxb = nx_bucket(nx);
    a.zs = take((size_t)batch * nx);
    a.vs = take((size_t)batch * nu);
    a.mus = take((size_t)batch * n);
    a.sgs = take((size_t)batch * n);
    double* rlo_s = take((size_t)batch * nx);
    double* rhi_s = take((size_t)batch * nx);
    a.rlo_s = rlo_s; a.rhi_s = rhi_s;
    a.z = z; a.v = v; a.r_lo = r_lo; a.r_hi = r_hi; a.certified = certified;
    a.thrust_c = thrust > 0.0 ? thrust * dyn->dt / dyn->m : 0.0;
    a.pad = pad;
    a.U = chain ? dyn->n_units : 0;
    // chains whose trajectory data fits in LDS: the whole causal pass in one launch
    int npos = 0, slots = 0, threads = 0;
    bool fold = false;
    const size_t lds = chain ? fp_chain_plan(nx, nu, dyn->n_units, N, batch, &npos, &slots, &threads, &fold) : 0;
    if (lds > 0) {
        FpChainArgs c = {};
        c.phi = phi; c.E = E; c.sigE = sigE; c.z = z; c.v = v;
        c.mu = mu; c.sigma = sigma; c.r_lo = r_lo; c.r_hi = r_hi; c.certified = certified;
        c.thrust_c = a.thrust_c;
        c.nu = nu; c.nw = nw; c.N = N; c.npos = npos; c.slots = slots;
        c.U = dyn->n_units;
        c.c = dyn->dt / dyn->m; c.kL = dyn->k_spring * dyn->rest_len; c.L0 = dyn->rest_len; c.pad = pad;
        const auto kern = fold ? sls_fp_chain_kernel<true> : sls_fp_chain_kernel<false>;
        if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SLS_LDS_MAX) !=
            hipSuccess)
            return LEB_EDEVICE;
        hipLaunchKernelGGL(kern, dim3((unsigned)batch), dim3((unsigned)threads), lds, s, c);
        return hipGetLastError() == hipSuccess ? LEB_OK : LEB_EDEVICE;
    }
    // otherwise one row launch and one bound launch per step
    for (int k = 0; k <= N; ++k) {
        const dim3 g((unsigned)batch), bl(SLS_THREADS);
        if (nxb == 8) hipLaunchKernelGGL(sls_fp_row_kernel<8>, g, bl, smem, s, a, k);
        else if (nxb == 16) hipLaunchKernelGGL(sls_fp_row_kernel<16>, g, bl, smem, s, a, k);
        else hipLaunchKernelGGL(sls_fp_row_kernel<32>, g, bl, smem, s, a, k);
        if (k == N) break;
        rc = chain ? launch_pbh_chain(dyn, batch, a.zs, a.vs, a.mus, a.sgs, rlo_s, rhi_s, nullptr, nullptr, 0.0,
                                      nullptr, s)
                   : launch_small_dyn(dyn, LEB_IH_PATH, batch, a.zs, a.vs, a.mus, a.sgs, rlo_s, rhi_s, nullptr,
                                      nullptr, 0.0, nullptr, s);
        if (rc) return rc;
    }
    return hipGetLastError() == hipSuccess ? LEB_OK : LEB_EDEVICE;
}
