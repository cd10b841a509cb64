// nn_hid.hpp -- CROWN passes of a ReLU MLP, shared by the bound (nn.hip) and its
// adjoint (nn_bwd.hip): the bounds of hidden layers 2 and 3 of networks with 16
// inputs, and the chain of any target layer.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "leb.h"
#include "leb_internal.hpp"
#include "nn_net.hpp"

namespace leb {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr double RT = 0x1p-40;   // rounding allowance factor of the bound

// ------------------------------------------- hidden targets, 16-wide input
//
// Both modes of one or two steps run in one workgroup.  In the first step Lambda is rows
// of W_k, the same for both modes, and on a neuron that is stably active (l >= 0)
// both modes multiply it by 1: those neurons' products are formed once and start
// both modes' accumulators; only the unstable neurons are multiplied per mode.
// Lists of the two classes (stably inactive neurons are in neither) are built per
// box.  The bounds are formed from the accumulators at the end (concretisation),
// so neither Lambda_0 nor its sums reach memory.
struct HidArgs {
    const double* WTt;             // target layer k, transposed: [w_{k-1}][M]
    const double* bt;              // [M]
    const double* W1; const double* W2;      // [w_1][16], [w_2][w_1]
    const double* b1; const double* b2;
    int w1, w2, M;
    // bounds of hidden layer 1 at lo, hi + box * bstride, of layer 2 at + lstride;
    // bound: slopes s, a, intercepts t, rounding weights e at the same offsets
    const double* lo; const double* hi;
    const double* s; const double* t; const double* a; const double* e;
    size_t bstride, lstride;
    const double* c; const double* rho;      // + box * cstride: [16]
    size_t cstride;
    double* lo_out; double* hi_out;          // + box * bstride: the target layer's bounds
    // adjoint: levels Lambda^(0) ([M][16] at off0) and Lambda^(1) ([M][w_1] at off1) of
    // direction d at lv + (2 box + d) lv_bm; validity of each box
    double* lv; size_t lv_bm; int off0, off1;
    const uint32_t* ok;
};

// ReLU relaxation of a neuron with pre-activation bounds [lo, hi] in exact
// arithmetic: upper line s z + t, lower line a z
__device__ __forceinline__ void nb_relax(double lo, double hi, double& s, double& t, double& a) {
    if (lo >= 0.0) { s = 1.0; t = 0.0; a = 1.0; }
    else if (hi > 0.0) { s = hi / (hi - lo); t = -s * lo; a = hi >= -lo ? 1.0 : 0.0; }
    else { s = 0.0; t = 0.0; a = 0.0; }
}

// neuron's relaxation and rounding weight at offset o (ADJ: none)
template <bool ADJ>
__device__ __forceinline__ void hid_relax(const HidArgs& A, size_t o, double l, double h, double& s, double& t,
                                          double& a, double& e) {
    if constexpr (ADJ) {
        nb_relax(l, h, s, t, a);
        e = 0.0;
    } else {
        s = A.s[o]; t = A.t[o]; a = A.a[o]; e = A.e[o];
    }
}

constexpr int HID_PAD = NN_MAXW + 12;        // listed neurons, padded past the last k-step read

// The two lists of one layer and the vectors their k-steps need, in list order.
struct HidLists {
    int na, nu;                              // active, unstable
    int ka[HID_PAD], ku[HID_PAD];
    double ab[HID_PAD], ae[HID_PAD];         // active: bias, rounding weight
    double us[HID_PAD], ua[HID_PAD], ut[HID_PAD], ub[HID_PAD], ue[HID_PAD];
};

// Built by 256 lanes (neuron `tid` of K <= 256) from the vectors at offset o; contains
// barriers.  A neuron with l >= 0 and u <= 0 has input 0 on the whole box: the bound
// drops it, the adjoint keeps it (its derivative is that of an active one).
template <bool ADJ>
__device__ __forceinline__ void hid_lists(HidLists& L, const HidArgs& A, size_t o, int K, const double* b,
                                          int (*cnt)[4]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool in = tid < K;
    const double l = in ? A.lo[o + tid] : -1.0, h = in ? A.hi[o + tid] : -1.0;
    const bool keep = h > 0.0 || (ADJ && l >= 0.0), act = keep && l >= 0.0, uns = keep && !act;
    const uint64_t ba = __ballot(act), bu = __ballot(uns), below = (1ull << lane) - 1ull;
    if (lane == 0) { cnt[0][wave] = __popcll(ba); cnt[1][wave] = __popcll(bu); }
    __syncthreads();
    int oa = 0, ou = 0, na = 0, nu = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        oa += q < wave ? cnt[0][q] : 0;
        ou += q < wave ? cnt[1][q] : 0;
        na += cnt[0][q];
        nu += cnt[1][q];
    }
    double s = 0.0, t = 0.0, a = 0.0, e = 0.0;
    if (keep) hid_relax<ADJ>(A, o + tid, l, h, s, t, a, e);
    if (act) {
        const int p = oa + __popcll(ba & below);
        L.ka[p] = tid;
        L.ab[p] = b[tid];
        L.ae[p] = e;
    }
    if (uns) {
        const int p = ou + __popcll(bu & below);
        L.ku[p] = tid;
        L.us[p] = s; L.ua[p] = a; L.ut[p] = t; L.ub[p] = b[tid]; L.ue[p] = e;
    }
    // twelve padding entries past each list (neuron 0, x forced to 0 by its readers)
    if (tid < 12) {
        L.ka[na + tid] = 0; L.ab[na + tid] = 0.0; L.ae[na + tid] = 0.0;
        L.ku[nu + tid] = 0;
        L.us[nu + tid] = L.ua[nu + tid] = L.ut[nu + tid] = L.ub[nu + tid] = L.ue[nu + tid] = 0.0;
    }
    if (tid == 0) { L.na = na; L.nu = nu; }
    __syncthreads();
}

// sum over the four lane groups of a 16 x 16 tile's columns
__device__ __forceinline__ double sum_groups(double x) {
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}

// The bound of target row `row` (lane column) in one mode from its Lambda_0^T tile
// (element i of lane group g: input 4 i + g) and its partial sums; the same in
// every lane group.
template <bool ADJ>
__device__ __forceinline__ double hid_concretize(const HidArgs& A, int box, int row, int mode, const d4& L0, double pb,
                                                 double pe, int g) {
    const double* c = A.c + (size_t)box * A.cstride;
    const double* rho = A.rho + (size_t)box * A.cstride;
    double lin = 0.0, mag = 0.0, ab = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double cn = c[4 * i + g], rn = rho[4 * i + g];
        lin = __builtin_fma(L0[i], cn, lin);
        mag = __builtin_fma(fabs(L0[i]), rn, mag);
        if (!ADJ) ab = __builtin_fma(fabs(L0[i]), fabs(cn), ab);
    }
    lin = sum_groups(lin); mag = sum_groups(mag); pb = sum_groups(pb);
    const double bt = row < A.M ? A.bt[row] : 0.0, beta = bt + pb;
    double err = 0.0;
    if (!ADJ) {
        ab = sum_groups(ab); pe = sum_groups(pe);
        err = RT * (pe + fabs(bt) + ab + mag + fabs(beta) + fabs(lin));
    }
    const double out = mode == 0 ? lin + mag + beta + err : lin - mag + beta - err;
    if (g == 0 && row < A.M) (mode == 0 ? A.hi_out : A.lo_out)[(size_t)box * A.bstride + row] = out;
    return out;
}

// adjoint: store row `row` of Lambda_0 of one direction
__device__ __forceinline__ void hid_store0(const HidArgs& A, int box, int row, int mode, const d4& L0, int g) {
    double* dst = A.lv + ((size_t)box * 2 + mode) * A.lv_bm + A.off0 + (size_t)row * 16 + g;
#pragma unroll
    for (int i = 0; i < 4; ++i) dst[4 * i] = L0[i];
}

// NT row tiles (wave, wave + 4, ...) of one wave: the products, then the bounds.
template <bool ADJ, int NT>
__device__ __forceinline__ void hid1_tiles(const HidArgs& A, const HidLists& L, int box, int wave, int r, int g) {
    const int na = L.na, nu = L.nu;
    const unsigned M8 = 8u * A.M;
    d4 U[NT], D[NT];
    double pb[NT], pbu[NT], pbl[NT], pe[NT];
#pragma unroll
    for (int q = 0; q < NT; ++q) {
        U[q] = d4{0.0, 0.0, 0.0, 0.0};
        pb[q] = pbu[q] = pbl[q] = pe[q] = 0.0;
    }
    double wn[2], xn[2][NT];                              // operands of two k-steps in flight
    auto fetch = [&](int p, int k, bool ok) {             // neuron k of this lane group
        const unsigned kx = __umul24(k, M8) + 8u * (16 * wave + r);
        wn[p] = A.W1[k * 16 + r];
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const double x = *(const double*)((const char*)A.WTt + (kx + 512u * q));
            xn[p][q] = ok ? x : 0.0;
        }
    };
    auto active = [&](int p, int c0) {
        const int c = c0 + g;
        const double w = wn[p], b = L.ab[c], e = L.ae[c];
        double x[NT];
#pragma unroll
        for (int q = 0; q < NT; ++q) x[q] = xn[p][q];
        fetch(p, L.ka[c + 8], c + 8 < na);                // past the end: padding
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            U[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(w, x[q], U[q], 0, 0, 0);
            pb[q] = __builtin_fma(x[q], b, pb[q]);
            if (!ADJ) pe[q] = __builtin_fma(fabs(x[q]), e, pe[q]);
        }
    };
    auto unstable = [&](int p, int c0) {
        const int c = c0 + g;
        const double w = wn[p], s = L.us[c], a = L.ua[c], t = L.ut[c], b = L.ub[c], e = L.ue[c];
        double x[NT];
#pragma unroll
        for (int q = 0; q < NT; ++q) x[q] = xn[p][q];
        fetch(p, L.ku[c + 8], c + 8 < nu);                // past the end: padding
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const bool pos = x[q] >= 0.0;
            const double xs = x[q] * s, xa = x[q] * a, xt = x[q] * t;
            const double ou = pos ? xs : xa, ol = pos ? xa : xs;
            U[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(w, ou, U[q], 0, 0, 0);
            D[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(w, ol, D[q], 0, 0, 0);
            pbu[q] = __builtin_fma(ou, b, pbu[q] + (pos ? xt : 0.0));
            pbl[q] = __builtin_fma(ol, b, pbl[q] + (pos ? 0.0 : xt));
            if (!ADJ) pe[q] = __builtin_fma(fabs(x[q]), e, pe[q]);
        }
    };
    fetch(0, L.ka[g], g < na);
    fetch(1, L.ka[g + 4], g + 4 < na);
    int c0 = 0;
    for (; c0 + 4 < na; c0 += 8) {
        active(0, c0);
        active(1, c0 + 4);
    }
    if (c0 < na) active(0, c0);
    fetch(0, L.ku[g], g < nu);
    fetch(1, L.ku[g + 4], g + 4 < nu);
#pragma unroll
    for (int q = 0; q < NT; ++q) D[q] = U[q];
    c0 = 0;
    for (; c0 + 4 < nu; c0 += 8) {
        unstable(0, c0);
        unstable(1, c0 + 4);
    }
    if (c0 < nu) unstable(0, c0);
#pragma unroll
    for (int q = 0; q < NT; ++q) {
        const int row = 16 * (wave + 4 * q) + r;
        const double h = hid_concretize<ADJ>(A, box, row, 0, U[q], pb[q] + pbu[q], pe[q], g);
        const double l = hid_concretize<ADJ>(A, box, row, 1, D[q], pb[q] + pbl[q], pe[q], g);
        // only an unstable neuron's rows are read back
        if (ADJ && l < 0.0 && h > 0.0) {
            hid_store0(A, box, row, 0, U[q], g);
            hid_store0(A, box, row, 1, D[q], g);
        }
    }
}

// Target layer 2: Lambda_0 = (W_2 (.) S_1) W_1, one workgroup per box; wave w owns the
// row tiles w, w + 4, ... (up to four) and runs all k-steps, so nothing is summed
// over waves.  A: W_1 rows of the listed neurons, B: the same rows of W_2^T.
//
// What bounds it: the operands' path from L2 (five reads a k-step for 4 or 8 MFMA).
// 3,200 boxes of the 16-256-256-256-12 network: 158 us with the concretisation
// (173 us with one k-step in flight and a branch per row tile; one workgroup per mode
// with its k-steps split over the waves: 690 us, and 42 us).
template <bool ADJ>
__global__ void __launch_bounds__(256) nn_hid1_kernel(HidArgs A) {
    __shared__ HidLists L;
    __shared__ int cnt[2][4];
    const int box = blockIdx.x, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (ADJ && !A.ok[box]) return;
    hid_lists<ADJ>(L, A, (size_t)box * A.bstride, A.w1, A.b1, cnt);
    // the loops for this wave's number of row tiles (no branch inside a k-step, so that
    // the waits on loads in flight are exact)
    const int nmine = ((A.M >> 4) - wave + 3) >> 2;
    if (nmine == 4) hid1_tiles<ADJ, 4>(A, L, box, wave, r, g);
    else if (nmine == 3) hid1_tiles<ADJ, 3>(A, L, box, wave, r, g);
    else if (nmine == 2) hid1_tiles<ADJ, 2>(A, L, box, wave, r, g);
    else if (nmine == 1) hid1_tiles<ADJ, 1>(A, L, box, wave, r, g);
}

// The first step of target layer 3 for one wave: NT tiles of 16 listed columns of W_2
// (byte offsets wcol8 of the lane's columns), two tiles of target rows (row8).  Two
// k-steps of operands are in flight.
template <bool ADJ, int NT>
__device__ __forceinline__ void hid2_first(const HidArgs& A, const HidLists& L, const unsigned (&wcol8)[4],
                                           const unsigned (&row8)[2], int first, int g, d4 (&U)[4][2], d4 (&D)[4][2],
                                           double (&pb)[2], double (&pbu)[2], double (&pbl)[2], double (&pe)[2]) {
    const int na = L.na, nu = L.nu;
    const unsigned N8 = 8u * A.w1, M8 = 8u * A.M;
    double wn[2][4], xn[2][2];
    auto fetch = [&](int p, int k, bool ok) {
        const unsigned kw = __umul24(k, N8), kx = __umul24(k, M8);
#pragma unroll
        for (int i = 0; i < NT; ++i) wn[p][i] = *(const double*)((const char*)A.W2 + (kw + wcol8[i]));
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const double x = *(const double*)((const char*)A.WTt + (kx + row8[q]));
            xn[p][q] = ok ? x : 0.0;
        }
    };
    auto active = [&](int p, int c0) {
        const int c = c0 + g;
        double w[4], x[2];
#pragma unroll
        for (int i = 0; i < NT; ++i) w[i] = wn[p][i];
#pragma unroll
        for (int q = 0; q < 2; ++q) x[q] = xn[p][q];
        fetch(p, L.ka[c + 8], c + 8 < na);                // past the end: padding
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int q = 0; q < 2; ++q) U[i][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[i], x[q], U[i][q], 0, 0, 0);
        if (((c0 >> 2) & 3) == first) {
            const double b = L.ab[c], e = L.ae[c];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                pb[q] = __builtin_fma(x[q], b, pb[q]);
                if (!ADJ) pe[q] = __builtin_fma(fabs(x[q]), e, pe[q]);
            }
        }
    };
    auto unstable = [&](int p, int c0) {
        const int c = c0 + g;
        double w[4], x[2], ou[2], ol[2];
#pragma unroll
        for (int i = 0; i < NT; ++i) w[i] = wn[p][i];
#pragma unroll
        for (int q = 0; q < 2; ++q) x[q] = xn[p][q];
        fetch(p, L.ku[c + 8], c + 8 < nu);                // past the end: padding
        const double s = L.us[c], a = L.ua[c];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const bool pos = x[q] >= 0.0;
            ou[q] = x[q] * (pos ? s : a);
            ol[q] = x[q] * (pos ? a : s);
        }
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                U[i][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[i], ou[q], U[i][q], 0, 0, 0);
                D[i][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[i], ol[q], D[i][q], 0, 0, 0);
            }
        if (((c0 >> 2) & 3) == first) {
            const double t = L.ut[c], b = L.ub[c], e = L.ue[c];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const double xt = x[q] * t;
                const bool pos = x[q] >= 0.0;
                pbu[q] = __builtin_fma(ou[q], b, pbu[q] + (pos ? xt : 0.0));
                pbl[q] = __builtin_fma(ol[q], b, pbl[q] + (pos ? 0.0 : xt));
                if (!ADJ) pe[q] = __builtin_fma(fabs(x[q]), e, pe[q]);
            }
        }
    };
    fetch(0, L.ka[g], g < na);
    fetch(1, L.ka[g + 4], g + 4 < na);
    int c0 = 0;
    for (; c0 + 4 < na; c0 += 8) {
        active(0, c0);
        active(1, c0 + 4);
    }
    if (c0 < na) active(0, c0);
    fetch(0, L.ku[g], g < nu);
    fetch(1, L.ku[g + 4], g + 4 < nu);
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int q = 0; q < 2; ++q) D[i][q] = U[i][q];
    c0 = 0;
    for (; c0 + 4 < nu; c0 += 8) {
        unstable(0, c0);
        unstable(1, c0 + 4);
    }
    if (c0 < nu) unstable(0, c0);
}

// Target layer 3, 32 of its rows and one box per workgroup: Lambda_1 = (W_3 (.) S_2) W_2
// in the columns of layer 1's neurons that are not stably inactive (the others are
// multiplied by 0 below), wave w owning every fourth tile of them, then Lambda_0 =
// (Lambda_1 (.) S_1) W_1.  The transposed accumulator of the first step (lane l holds
// neuron [4 i + l/16] of row [l%16]) is the B operand of the second, so each wave
// multiplies its own tiles' neurons straight from its registers and only the four
// waves' 16 x 16 partial tiles meet in LDS.  Row sums of the first step are taken
// by the waves in turn (k-step modulo 4).
//
// What bounds it: FP64 MFMA (about 1,000 a workgroup of the 16-256-256-256-12
// network where both modes over all kept neurons and every column took 2,416: 0.7 ms
// at the peak rate) and the latency of the operand reads from L2, two waves a SIMD.
// 3,200 boxes: 1.37 ms, the adjoint's 1.50 ms (one k-step in flight, and branches on
// the tiles in each: 1.76 ms; eight waves of half the tiles each, four a SIMD: the
// same 1.77; every column of Lambda_1: 2.12 ms; one workgroup per mode and 16 rows with Lambda in LDS between the steps: 4.2 ms,
// and 42 us to concretise; the adjoint's general pass 6.4 ms).
template <bool ADJ>
__global__ void __launch_bounds__(256, 2) nn_hid2_kernel(HidArgs A) {
    __shared__ HidLists L;
    // layer 1: the neurons that are not stably inactive (the columns of Lambda_1 that
    // are formed), padded to whole tiles, and their s, a, t, bias, e (0 in the padding)
    __shared__ int col1[NN_MAXW];
    __shared__ double v1[5][NN_MAXW];
    __shared__ double part[4][4][4][64];                  // waves: partial tiles (row tile, mode)
    __shared__ double psum[4][4][2][64];                  // waves: bias and rounding sums (row tile, mode)
    __shared__ int cnt[2][4], cnt1[4];
    const int box = blockIdx.y, row0 = 32 * blockIdx.x, tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (ADJ && !A.ok[box]) return;
    const size_t o1 = (size_t)box * A.bstride, o2 = A.lstride + o1;
    const int M = A.M, N = A.w1;
    int n1 = 0;
    {
        const double l = tid < N ? A.lo[o1 + tid] : -1.0, h = tid < N ? A.hi[o1 + tid] : -1.0;
        const bool keep = h > 0.0 || (ADJ && l >= 0.0);
        const uint64_t bal = __ballot(keep);
        if (lane == 0) cnt1[wave] = __popcll(bal);
        double s = 0.0, t = 0.0, a = 0.0, e = 0.0;
        if (keep) hid_relax<ADJ>(A, o1 + tid, l, h, s, t, a, e);
        col1[tid] = 0;
#pragma unroll
        for (int q = 0; q < 5; ++q) v1[q][tid] = 0.0;
        __syncthreads();
        int off = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            off += q < wave ? cnt1[q] : 0;
            n1 += cnt1[q];
        }
        if (keep) {
            const int p = off + __popcll(bal & ((1ull << lane) - 1ull));
            col1[p] = tid;
            v1[0][p] = s; v1[1][p] = a; v1[2][p] = t; v1[3][p] = A.b1[tid]; v1[4][p] = e;
        }
    }
    hid_lists<ADJ>(L, A, o2, A.w2, A.b2, cnt);
    // this wave's tiles of the listed columns: first, first + 4, ... (first rotates over
    // the workgroups, so that the waves with a tile more spread over the SIMDs; every sum
    // below is split and added by `first`, so that a box's result does not depend on its place)
    const int na = L.na, nu = L.nu, nt = (n1 + 15) >> 4;
    const int first = (wave + blockIdx.x + blockIdx.y) & 3, nmine = (nt - first + 3) >> 2;
    d4 U[4][2], D[4][2];
    double pb[2] = {0.0, 0.0}, pbu[2] = {0.0, 0.0}, pbl[2] = {0.0, 0.0}, pe[2] = {0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < 2; ++q) U[i][q] = d4{0.0, 0.0, 0.0, 0.0};
    // first step, the loops for this wave's number of tiles (no branch inside a k-step,
    // so that the waits on loads in flight are exact)
    unsigned wcol8[4], row8[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) wcol8[i] = 8u * col1[i < nmine ? 16 * (first + 4 * i) + r : 0];
#pragma unroll
    for (int q = 0; q < 2; ++q) row8[q] = 8u * (row0 + 16 * q < M ? row0 + 16 * q + r : row0 + r);
    if (nmine == 4) hid2_first<ADJ, 4>(A, L, wcol8, row8, first, g, U, D, pb, pbu, pbl, pe);
    else if (nmine == 3) hid2_first<ADJ, 3>(A, L, wcol8, row8, first, g, U, D, pb, pbu, pbl, pe);
    else if (nmine == 2) hid2_first<ADJ, 2>(A, L, wcol8, row8, first, g, U, D, pb, pbu, pbl, pe);
    else if (nmine == 1) hid2_first<ADJ, 1>(A, L, wcol8, row8, first, g, U, D, pb, pbu, pbl, pe);
    else hid2_first<ADJ, 0>(A, L, wcol8, row8, first, g, U, D, pb, pbu, pbl, pe);
    // second step: this wave's listed neurons 16 tt + 4 j + g of layer 1
    d4 Z[2][2];                                           // (row tile, mode): Lambda_0^T
    double sb[2][2], se[2][2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        sb[q][0] = pb[q] + pbu[q]; sb[q][1] = pb[q] + pbl[q];
        se[q][0] = se[q][1] = pe[q];
        Z[q][0] = Z[q][1] = d4{0.0, 0.0, 0.0, 0.0};
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i >= nmine) break;
        const int n0 = 16 * (first + 4 * i) + g;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = n0 + 4 * j;
            const double w = A.W1[col1[n] * 16 + r];
            const double s = v1[0][n], a = v1[1][n], t = v1[2][n], b = v1[3][n], e = v1[4][n];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const double xu = U[i][q][j], xl = D[i][q][j];
                const bool pu = xu >= 0.0, pl = xl >= 0.0;
                const double ou = xu * (pu ? s : a), ol = xl * (pl ? a : s);
                Z[q][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(w, ou, Z[q][0], 0, 0, 0);
                Z[q][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(w, ol, Z[q][1], 0, 0, 0);
                sb[q][0] = __builtin_fma(ou, b, sb[q][0] + (pu ? xu * t : 0.0));
                sb[q][1] = __builtin_fma(ol, b, sb[q][1] + (pl ? 0.0 : xl * t));
                if (!ADJ) {
                    se[q][0] = __builtin_fma(fabs(xu), e, se[q][0]);
                    se[q][1] = __builtin_fma(fabs(xl), e, se[q][1]);
                }
            }
        }
    }
    // the waves' partial tiles and sums; wave w finishes (row tile w / 2, mode w % 2)
#pragma unroll
    for (int m = 0; m < 4; ++m) {
#pragma unroll
        for (int i = 0; i < 4; ++i) part[first][m][i][lane] = Z[m >> 1][m & 1][i];
        psum[first][m][0][lane] = sb[m >> 1][m & 1];
        psum[first][m][1][lane] = se[m >> 1][m & 1];
    }
    __syncthreads();
    d4 z = d4{0.0, 0.0, 0.0, 0.0};
    double b = 0.0, e = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
#pragma unroll
        for (int i = 0; i < 4; ++i) z[i] += part[w][wave][i][lane];
        b += psum[w][wave][0][lane];
        e += psum[w][wave][1][lane];
    }
    const int row = row0 + 16 * (wave >> 1) + r;
    const double v = hid_concretize<ADJ>(A, box, row, wave & 1, z, b, e, g);
    if constexpr (ADJ) {
        // only an unstable neuron's rows are read back: both directions' bounds meet in LDS
        __syncthreads();                                  // part and psum read
        if (g == 0) psum[0][wave & 1][0][16 * (wave >> 1) + r] = row < M ? v : 0.0;
        __syncthreads();
        bool uns[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) uns[q] = psum[0][1][0][16 * q + r] < 0.0 && psum[0][0][0][16 * q + r] > 0.0;
        if (uns[wave >> 1]) hid_store0(A, box, row, wave & 1, z, g);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i >= nmine) break;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = 16 * (first + 4 * i) + 4 * j + g;
                if (n >= n1) continue;
                double* dst = A.lv + (size_t)box * 2 * A.lv_bm + A.off1 + (size_t)(row0 + r) * N + col1[n];
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (uns[q]) {
                        dst[(size_t)16 * q * N] = U[i][q][j];
                        dst[A.lv_bm + (size_t)16 * q * N] = D[i][q][j];
                    }
            }
        }
    }
}

// ---------------------------------------------------------- 16 boxes a workgroup
//
// A layer's products for 16 boxes (the forms of nn.hip and nn_bwd.hip for many boxes).
constexpr int NNG_BOXES = 16, NNG_T = 512, NNG_RS = 17;     // boxes, lanes, LDS row stride
constexpr int NNG_MIN = 1024;                               // fewest boxes for the grouped form

// Y[c][n][box] for the output tiles t = wave, wave + 8 (acc[q][c]): chain 0 by W (SIGNED, else by
// |W|), the others by |W|; inputs X[c][k][box], RELU: of the neurons with X[0] > 0 (chains 0 and 2).
template <int NC, bool SIGNED, bool RELU>
__device__ __forceinline__ void group_products(const double* WT, int in, int out, const double* X, int wave, int r,
                                               int g, d4 (&acc)[2][NC]) {
    const int nt = (out + 15) >> 4;                          // a ragged last tile repeats its last output
    if (wave >= nt) return;
    const int t1 = wave + 8 < nt ? wave + 8 : wave;
    const double* w0 = WT + (size_t)g * out + min(16 * wave + r, out - 1);
    const double* w1 = WT + (size_t)g * out + min(16 * t1 + r, out - 1);
    double wn[2][2];
#pragma unroll
    for (int p = 0; p < 2; ++p) { wn[p][0] = w0[(size_t)4 * p * out]; wn[p][1] = w1[(size_t)4 * p * out]; }
    for (int s = 0; s < in >> 2; s += 2) {                  // widths are multiples of 16
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            double x[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) x[c] = X[(c * NN_MAXW + 4 * (s + p) + g) * NNG_RS + r];
            if (RELU) {
                const bool on = x[0] > 0.0;
                x[0] = on ? x[0] : 0.0;
                if (NC > 2) x[NC - 1] = on ? x[NC - 1] : 0.0;
            }
            const double a0 = wn[p][0], a1 = wn[p][1];
            const size_t o = (size_t)4 * (s + p + 2 < in >> 2 ? s + p + 2 : s + p) * out;
            wn[p][0] = w0[o];
            wn[p][1] = w1[o];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                acc[0][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(c == 0 && SIGNED ? a0 : fabs(a0), x[c], acc[0][c], 0, 0, 0);
                acc[1][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(c == 0 && SIGNED ? a1 : fabs(a1), x[c], acc[1][c], 0, 0, 0);
            }
        }
    }
}


// ---------------------------------------------------------- fused chain
//
// The whole backward substitution of one target layer k, for one box, one
// mode and a block of 16 target rows, in one workgroup:
//   Lambda_{j-1} = (Lambda_j (.) S_j) W_j,   j = k-1, ..., 1,   Lambda_k = rows of W_k,
//   beta += sum_i (Lambda_j t_sel)_i + (Omega_j b_j),   eps += |Lambda_j| e_j,
// with Lambda kept in LDS between the steps (never in HBM).  Modes: 0 upper, 1
// lower, 2 Jacobian (S = 1[z^ > 0]).  The product is formed transposed on FP64
// MFMA (v_mfma_f64_16x16x4): Lambda^T_{j-1} = W_j^T Omega^T, so the accumulator of
// one step (lane l holds element [4i + l/16][l%16] of a 16 x 16 tile) is stored to
// LDS in the layout the next step reads its B operand from (lane l supplies
// B[l/16][l%16]).  A operands are W_j columns read from L2.
// The neurons of layer j with slope 0 in the mode (stably inactive; z^ <= 0 in the
// Jacobian) are listed out: a step runs over the other neurons only, and forms only
// their columns for the next step; the state sits at list positions.
// Wave w produces the output tiles w, w + 4, ... of each step; with one or two
// tiles the waves split the k-steps instead (partial tiles added in slice order).
//
// What bounds it: FP64 MFMA, three workgroups a compute unit hiding the L2 reads and
// the barriers between the steps.  Output pass of the 16-256-256-256-12 network, three
// modes, 3,200 boxes: 475 us (every column of Lambda formed, one k-step in flight:
// 740 us); 40 boxes of 16-128-128-128-12: 17 us (22 us).  The adjoint's output pass
// with the Jacobian's rows: 469 us (in the general pass: 680 us and, in its reverse
// launch, another 660 us for the Jacobian).
struct ChainArgs {
    const double* WTt;             // target layer k, transposed: [w_{k-1}][M] (shared by every box)
    const double* bt;              // [M]
    const double* W[NN_MAXL];      // layer j at W[j-1]: [w_j][w_{j-1}]
    const double* b[NN_MAXL];
    int w[NN_MAXL + 1];
    int k, M, nbox;
    // per-box vectors of hidden layer j (1-based) at base + (j - 1) * lstride + box * bstride
    // (adjoint: the bounds only); D (adjoint: z^) with strides of its own
    const double* lo; const double* hi;
    const double* s; const double* t; const double* a; const double* e; const double* D;
    size_t bstride, lstride, dbstride, dlstride;
    double* C;                     // bound: [mode][box][M][w_0]
    double* beta; double* eps;     // bound: [mode][box][M]
    // adjoint: levels j = 0 .. k - 2 of mode 0, 1 at lv + (2 box + mode) lv_bm + off[j], [M][w_j];
    // the Jacobian's rows at jac + box * jstride, [M][w_0]
    double* lv; size_t lv_bm; int off[NN_MAXL];
    double* jac; size_t jstride;
    const uint32_t* ok;
};

constexpr size_t CHAIN_STATE_BYTES = (size_t)NN_MAXW * 16 * sizeof(double);
constexpr int CHAIN_PAD = NN_MAXW + 8;               // listed neurons, padded past the last k-step read
constexpr int CHAIN_PAD2 = NN_MAXW + 40;             // ... and past the last k-step fetched ahead

struct ChainLists {
    double v[5][CHAIN_PAD];        // slope x >= 0, slope x < 0, intercept, bias, e (list order)
    int k[2][CHAIN_PAD2];          // listed neurons of the step's layer and of the layer below
};

// The k-loop of one step for one wave: NT tiles of output columns (col8: byte offsets
// of the lane's columns in a row of W), k-steps 4 slice, 4 slice + 4 nslice, ... of the
// list; x of the rows from W_k^T (FIRST) or from the state in LDS.
template <bool FIRST, bool SUMS, int NT>
__device__ __forceinline__ void chain_steps(const double* W, unsigned N8, const double* WTt, unsigned M8, unsigned row8,
                                            const double* cst, const ChainLists& L, const int* kl, int Kc,
                                            const unsigned (&col8)[4], int slice, int nslice, int turn, int g, int r,
                                            bool t_on_pos, bool t_on_neg, d4 (&acc)[4], double& pb, double& pe) {
    double wn[2][4], xn[2];
    const int stride = 4 * nslice;
    auto fetch = [&](int p, int c) {
        const unsigned k = kl[c];
        const unsigned kw = __umul24(k, N8);
#pragma unroll
        for (int i = 0; i < NT; ++i) wn[p][i] = *(const double*)((const char*)W + (kw + col8[i]));
        double x;
        if (FIRST) x = *(const double*)((const char*)WTt + (__umul24(k, M8) + row8));
        else x = cst[(c < NN_MAXW ? c : 0) * 16 + r];
        xn[p] = c < Kc ? x : 0.0;
    };
    auto step = [&](int p, int c0, int n) {
        const int c = c0 + g;
        double w[4];
#pragma unroll
        for (int i = 0; i < NT; ++i) w[i] = wn[p][i];
        const double x = xn[p];
        fetch(p, c + 2 * stride);                         // past the end: padding
        const bool pos = x >= 0.0;
        const double om = x * (pos ? L.v[0][c] : L.v[1][c]);
#pragma unroll
        for (int i = 0; i < NT; ++i) acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[i], om, acc[i], 0, 0, 0);
        if (SUMS && (turn < 0 || (n & 3) == turn)) {
            const double xt = x * L.v[2][c];
            pb = __builtin_fma(om, L.v[3][c], pb + ((pos ? t_on_pos : t_on_neg) ? xt : 0.0));
            pe = __builtin_fma(fabs(x), L.v[4][c], pe);
        }
    };
    int c0 = 4 * slice, n = 0;
    if (c0 >= Kc) return;
    fetch(0, c0 + g);
    fetch(1, c0 + stride + g);
    for (; c0 + stride < Kc; c0 += 2 * stride, n += 2) {
        step(0, c0, n);
        step(1, c0 + stride, n + 1);
    }
    if (c0 < Kc) step(0, c0, n);
}

template <bool ADJ>
__global__ void __launch_bounds__(256, 3) nn_chain_kernel(ChainArgs A) {
    extern __shared__ double cst[];                    // [list position or input][16]: Lambda^T of this block
    __shared__ ChainLists L;
    __shared__ int scnt[4];
    __shared__ double spart[768];                      // partial tiles of the k-slices; then the row sums
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int mode = blockIdx.y, box = blockIdx.z;
    if (ADJ && !A.ok[box]) return;
    // intercept of the selected line: upper mode on x >= 0, lower mode on x < 0
    const bool t_on_pos = mode == 0, t_on_neg = mode == 1;
    // list the neurons of layer j with a slope in this mode into L.k[p] and keep this
    // lane's neuron's vectors and list position in registers until stage() (the list
    // of the step above is still in use)
    int Kc = 0, pos_ = -1;
    double vr[5];
    auto prepare = [&](int j, int p) {
        const int K = A.w[j];
        const size_t o = (size_t)(j - 1) * A.lstride + (size_t)box * A.bstride + tid;
        bool keep = false;
#pragma unroll
        for (int q = 0; q < 5; ++q) vr[q] = 0.0;
        if (tid < K) {
            if (mode == 2) {
                keep = A.D[(size_t)(j - 1) * A.dlstride + (size_t)box * A.dbstride + tid] > 0.0;
                vr[0] = vr[1] = 1.0;
            } else {
                const double l = A.lo[o], h = A.hi[o];
                double s_, t_, a_, e_ = 0.0;
                keep = h > 0.0 || (ADJ && l >= 0.0);
                if (ADJ) nb_relax(l, h, s_, t_, a_);
                else { s_ = A.s[o]; t_ = A.t[o]; a_ = A.a[o]; e_ = A.e[o]; }
                vr[0] = mode == 0 ? s_ : a_;
                vr[1] = mode == 0 ? a_ : s_;
                vr[2] = t_;
                vr[4] = e_;
            }
            vr[3] = ADJ ? 0.0 : A.b[j - 1][tid];
        }
        const uint64_t bal = __ballot(keep);
        if (lane == 0) scnt[wave] = __popcll(bal);
        __syncthreads();
        int off = 0;
        Kc = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) { off += q < wave ? scnt[q] : 0; Kc += scnt[q]; }
        pos_ = keep ? off + __popcll(bal & ((1ull << lane) - 1ull)) : -1;
        if (keep) L.k[p][pos_] = tid;
        if (tid >= Kc) L.k[p][tid] = 0;                // padding (its x is forced to 0)
        if (tid < CHAIN_PAD2 - 256) L.k[p][256 + tid] = 0;
        __syncthreads();
    };
    auto stage = [&]() {                               // the vectors, in list order (0 in the padding)
        if (pos_ >= 0) {
#pragma unroll
            for (int q = 0; q < 5; ++q) L.v[q][pos_] = vr[q];
        }
        if (tid < 8) {
#pragma unroll
            for (int q = 0; q < 5; ++q) L.v[q][Kc + tid] = 0.0;
        }
    };
    const int M = A.M;
    // a target with one step (k = 2) runs every 16-row block in this workgroup with
    // one list; deeper targets run one block per workgroup
    const bool single = A.k == 2;
    const int nrb = (M + 15) / 16;
    int buf = 0;
    for (int rb = single ? 0 : blockIdx.x; rb < (single ? nrb : blockIdx.x + 1); ++rb) {
        const int row0 = 16 * rb;
        if (!single || rb == 0) {
            prepare(A.k - 1, buf);
            stage();
        }
        __syncthreads();
        double pb = 0.0, pe = 0.0;
        for (int j = A.k - 1; j >= 1; --j) {
            const int N = A.w[j - 1], kc = Kc;
            const int* kl = L.k[buf];
            int ncol = N;
            if (j > 1) {
                prepare(j - 1, buf ^ 1);               // columns of the layer below (registers until stage())
                ncol = Kc;
            }
            // work split: ntile >= 3: wave w owns tiles w, w + 4, ... over all k; ntile 2 or
            // 1: the waves split the k-steps of the tile(s) into 2 or 4 slices
            const int ntile = (ncol + 15) >> 4;
            const int nslice = ntile >= 3 || ntile == 0 ? 1 : 4 / ntile;
            const int slice = wave / (4 / nslice);
            const int tfirst = ntile >= 3 ? wave : (ntile == 2 ? wave & 1 : 0);
            const int nmine = ntile >= 3 ? (ntile - wave + 3) >> 2 : (ntile > 0 ? 1 : 0);
            // row sums: k-steps in turn over the waves, or each slice's by the wave of its first tile
            const int turn = nslice == 1 ? wave : (tfirst == 0 ? -1 : 4);
            d4 acc[4];
            unsigned col8[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[i] = d4{0.0, 0.0, 0.0, 0.0};
                const int c = i < nmine ? 16 * (tfirst + 4 * i) + r : 0;
                col8[i] = 8u * (j > 1 ? L.k[buf ^ 1][c] : c);
            }
            const unsigned N8 = 8u * N, M8 = 8u * M, row8 = 8u * min(row0 + r, M - 1);
            auto run = [&](auto first, auto nt) {
                chain_steps<decltype(first)::value, !ADJ, decltype(nt)::value>(
                    A.W[j - 1], N8, A.WTt, M8, row8, cst, L, kl, kc, col8, slice, nslice, turn, g, r, t_on_pos, t_on_neg,
                    acc, pb, pe);
            };
            using T_ = std::integral_constant<bool, true>;
            using F_ = std::integral_constant<bool, false>;
#define CHAIN_NT(F)                                                      \
    if (nmine == 4) run(F{}, std::integral_constant<int, 4>{});          \
    else if (nmine == 3) run(F{}, std::integral_constant<int, 3>{});     \
    else if (nmine == 2) run(F{}, std::integral_constant<int, 2>{});     \
    else if (nmine == 1) run(F{}, std::integral_constant<int, 1>{});     \
    else run(F{}, std::integral_constant<int, 0>{});
            if (j == A.k - 1) { CHAIN_NT(T_) } else { CHAIN_NT(F_) }
#undef CHAIN_NT
            // slices 1.. hand their partial tiles to slice 0 (added in slice order); every
            // read of the state and of the vectors is done before they are overwritten
            const int pidx = nslice == 4 ? slice - 1 : tfirst;
            if (nslice > 1 && slice > 0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) spart[pidx * 256 + q * 64 + lane] = acc[0][q];
            }
            __syncthreads();
            if (nslice > 1 && slice == 0) {
                for (int sl = 1; sl < nslice; ++sl) {
                    const int pi = nslice == 4 ? sl - 1 : tfirst;
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[0][q] += spart[pi * 256 + q * 64 + lane];
                }
            }
            if (j > 1) stage();
            if (slice == 0) {
                double* lv = ADJ && mode < 2 ? A.lv + ((size_t)box * 2 + mode) * A.lv_bm + A.off[j - 1] : nullptr;
                if (ADJ && j == 1 && mode == 2) lv = A.jac + (size_t)box * A.jstride;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (i >= nmine) break;
                    const int tt = tfirst + 4 * i;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int c = 16 * tt + 4 * q + g;
                        if (!ADJ || j > 1) cst[c * 16 + r] = acc[i][q];
                        if (ADJ && lv && c < ncol && row0 + r < M)
                            lv[(size_t)(row0 + r) * N + (j > 1 ? L.k[buf ^ 1][c] : c)] = acc[i][q];
                    }
                }
            }
            __syncthreads();                           // the next step reads the state just written
            if (j > 1) buf ^= 1;
        }
        if (!ADJ) {
            // Lambda_0 rows of this block, and the bias and rounding sums of each row
            const int n0 = A.w[0];
            const size_t cbase = ((size_t)mode * A.nbox + box) * M;
            for (int q = tid; q < 16 * n0; q += 256) {
                const int rr = q / n0, n = q - rr * n0;
                if (row0 + rr < M) A.C[(cbase + row0 + rr) * n0 + n] = cst[n * 16 + rr];
            }
            spart[wave * 64 + lane] = pb;
            spart[256 + wave * 64 + lane] = pe;
            __syncthreads();
            if (tid < 16 && row0 + tid < M) {
                double b_ = 0.0, e_ = 0.0;
                for (int w = 0; w < 4; ++w)
                    for (int q = 0; q < 4; ++q) { b_ += spart[w * 64 + tid + 16 * q]; e_ += spart[256 + w * 64 + tid + 16 * q]; }
                const double bt = A.bt[row0 + tid];
                A.beta[cbase + row0 + tid] = bt + b_;
                A.eps[cbase + row0 + tid] = e_ + fabs(bt);
            }
            __syncthreads();                           // the next block reuses the state and sums
        }
    }
}

template <bool ADJ>
static int launch_nn_chain(const ChainArgs& c, int nmode, int nact, hipStream_t st) {
    static DynLds lds;
    if (int rc = lds.raise((const void*)nn_chain_kernel<ADJ>, CHAIN_STATE_BYTES)) return rc;
    const unsigned rbs = c.k == 2 ? 1u : (unsigned)((c.M + 15) / 16);
    hipLaunchKernelGGL(nn_chain_kernel<ADJ>, dim3(rbs, nmode, nact), dim3(256), CHAIN_STATE_BYTES, st, c);
    return hipGetLastError() == hipSuccess ? LEB_OK : LEB_EDEVICE;
}

}  // namespace leb
