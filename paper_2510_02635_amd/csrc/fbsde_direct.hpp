// Direct solve of a level's ridge regression where one side of the design is small (Sec. 2.4, the normal
// equations (D'^T W D' + lambda I) alpha_x = D'^T W (Y - Ybar) with D'_j = s (W_j - Wbar)):
//   dual    (M <= d + 1, M <= FBSDE_DUAL_MAXM): alpha_x = B^T (B B^T + lambda I)^{-1} W^1/2 (Y - Ybar) with
//           B = W^1/2 D' (M x d), the push-through identity: one M x M system per point;
//   primal  (M > d + 1, d <= DIRECT_MAXD): (B^T B + lambda I) alpha_x = b, one d x d system per point.
// The matrix-free CG reads the cloud once per iteration, dozens of times a level in FP64; here it is read
// once, for the Gram matrix on the FP64 matrix cores (FP64 arithmetic on either state).
//   k_gram          partial Gram matrices over slices of the contraction (coordinates for the dual form,
//                   particles for the primal one), in 16 x 16 tiles of the upper triangle (fbsde_gram.hpp);
//   k_direct_fold   the slices' partials summed in order;
//   k_direct_solve  one block per point: factorisation and solution in registers (fbsde_spd.hpp);
//   k_direct_alpha  dual form: alpha_x = s sum_j w_j^1/2 c_j (W_j - Wbar) over the cloud.
// The result goes where the CG iterate goes, at the scale k_moments_finish chose, so the level's finish is the
// same.
#pragma once
#include "fbsde.h"
#include "fbsde_gram.hpp"

namespace fbsde {

// part[p][0][.] = sum over the slices, in order; grid (elements / 256, P).
__global__ void __launch_bounds__(256)
k_direct_fold(double* __restrict__ part, int nsplit, int64_t n) {
    const int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (e >= n) return;
    double* q = part + (int64_t)blockIdx.y * nsplit * n + e;
    double a = 0.0;
#pragma unroll 8
    for (int i = 0; i < nsplit; ++i) a += q[i * n];
    q[0] = a;
}

// Factors and solves the system of point blockIdx.x (n unknowns, the slices in `part` already folded: the point's matrix
// is at p * pstride, laid out by gram_index).  Dual: the right-hand side W^1/2 (Y - Ybar) at the
// level's scale; out: coef[p][j] = s w_j^1/2 c_j and coef[p][M] their sum.  Primal: right-hand side r, the
// slope goes to x.
template <int T, bool PRIMAL>
__global__ void __launch_bounds__(64 * spd_waves(T), spd_occupancy(T))
k_direct_solve(const double* __restrict__ part, int64_t pstride, int n, int ld, double s,
               const double* __restrict__ w, const double* __restrict__ Y, const double* __restrict__ r,
               const double* __restrict__ scal, int ns, double* __restrict__ coef, double* __restrict__ x,
               int* __restrict__ iscal, uint32_t* __restrict__ status) {
    constexpr int NW = spd_waves(T), BS = 64 * NW;
    __shared__ SpdShared<T> sh;
    __shared__ double bv[16 * T];
    __shared__ double red[16];
    const int p = blockIdx.x, t = threadIdx.x;
    const double* A = part + (int64_t)p * pstride;
    const double lam = scal[(int64_t)p * ns + 3];
    SpdSystem<T> sys;
    sys.init(blockIdx.x);
    bool any = false;
    if constexpr (PRIMAL) {
        for (int i = t; i < 16 * T; i += BS) {
            bv[i] = (i < n) ? r[(int64_t)p * ld + i] : 0.0;
            any |= bv[i] != 0.0;
        }
    } else {
        const double yb = scal[(int64_t)p * ns + 4], isc = scal[(int64_t)p * ns + 9];
        for (int i = t; i < 16 * T; i += BS) {
            bv[i] = (i < n) ? sqrt(w[(int64_t)p * n + i]) * (Y[(int64_t)p * n + i] - yb) / isc : 0.0;
            any |= bv[i] != 0.0;
        }
    }
    bool good = true;
    if (__syncthreads_or(any)) {
        const int np = spd_pivots(n);
        const uint32_t last = (uint32_t)(gram_entries(n) - 1);   // the padding reads some entry and takes zero
        good = sys.solve(
            [&](int i, int j) { return A[min((uint32_t)gram_index(n, i, j), last)]; },
            [&](double a, int i, int j) { return (max(i, j) < n) ? a : 0.0; }, [&](int i) { return (i < n) ? lam : 1.0; },
            [&](int i) { return bv[i]; }, np, np, sh);
    } else {   // as the CG: no step from zero, also where the cloud has no spread and the system is zero
        for (int i = t; i < 16 * T; i += BS) sh.x[i] = 0.0;
        __syncthreads();
    }
    if (!good && sys.lane == 0) atomicOr(&status[p], (uint32_t)ST_NONFINITE);
    if constexpr (PRIMAL) {
        for (int i = t; i < ld; i += BS) x[(int64_t)p * ld + i] = (i < n) ? sh.x[i] : 0.0;
    } else {
        double cs = 0.0;
        for (int j = t; j < n; j += BS) {
            const double cj = s * sqrt(w[(int64_t)p * n + j]) * sh.x[j];
            coef[(int64_t)p * (n + 1) + j] = cj;
            cs += cj;
        }
        cs = block_sum(cs, red);
        if (t == 0) coef[(int64_t)p * (n + 1) + n] = cs;
    }
    if (t == 0) {
        iscal[p * 4 + 0] = 0;   // no CG iterations
        iscal[p * 4 + 1] = 1;
    }
}

// alpha_x of the dual form: block (x, p) owns 64 coordinates, its four waves a quarter of the particles each.
template <typename S>
__global__ void __launch_bounds__(256)
k_direct_alpha(const double* __restrict__ coef, int M, const S* __restrict__ W, int64_t ldw, int ld,
               const double* __restrict__ Wbar, double* __restrict__ x) {
    __shared__ double cf[FBSDE_DUAL_MAXM];
    __shared__ double red[4][64];
    const int p = blockIdx.y, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int i = blockIdx.x * 64 + lane;
    const double* cp = coef + (int64_t)p * (M + 1);
    for (int j = t; j < M; j += 256) cf[j] = cp[j];
    __syncthreads();
    const int per = (M + 3) / 4, j0 = wv * per, j1 = min(M, j0 + per);
    double a = 0.0;
    if (i < ld) {
        const S* Wp = W + (int64_t)p * M * ldw + i;
#pragma unroll 8
        for (int j = j0; j < j1; ++j) a = fma(cf[j], (double)Wp[(int64_t)j * ldw], a);
    }
    red[wv][lane] = a;
    __syncthreads();
    if (wv == 0 && i < ld)
        x[(int64_t)p * ld + i] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane] -
                                 cp[M] * Wbar[(int64_t)p * ld + i];
}

}  // namespace fbsde
