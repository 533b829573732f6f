// Paper-literal per-anchor scheme on gfx950: Algorithm 1 as printed (Sec. 2.3 to 2.5), with one
// weighted ridge regression per particle m and level k. Each regression is set in X_k-space about
// the particle itself (eq. Dj, D^m_j = X^j_k - X^m_k) and penalises the intercept as printed. The
// conditional expectation is the plain particle mean (eq. discreteYkm).
//
// Per level and evaluation point, where W are the Brownian displacements and X = x0 + mu t + s W:
//   1. reversal    W_k = W_{k+1} - sqrt(dt) xi_k, with the increments regenerated from their counters
//                  (all particles start at x0, so W_0 = 0 exactly);
//   2. Gram        G = W_k W_k^T [M][M] and the row sums rho_j = sum_i W^j_k,i. Every anchor's
//                  design follows from them:
//                  D^m_i . D^m_j = s^2 (G_ij - G_im - G_jm + G_mm);
//   3. anchors     one block per (m, p). The ridge minimiser alpha = (alpha, alpha_x) of J_lambda
//                  comes from the M x M dual system (push-through identity):
//                    S = Om (1 1^T + K) Om + lambda I,  Om = diag(sqrt(w)),  K_ij = D_i . D_j,
//                    c = Om S^{-1} Om Y_{k+1},  alpha = sum_j c_j,  alpha_x = sum_j c_j D_j.
//                  S, bordered by the right-hand side Om Y as an extra column, is factored and solved
//                  in registers on the FP64 matrix cores (fbsde_spd.hpp). The nonlinearity needs only
//                  |Z|^2 = s^2 c^T K c and sum_i Z_i = s^2 sum_j c_j (rho_j - rho_m) (Z = s alpha_x).
//                  Both come from G without forming alpha_x. Newton (eq. NRiter) on
//                  y - Ybar - dt f(y, Z) then gives Y^m_k.
// Cost per level and point: O(M^2 d) for the Gram, and O(M^3 / 3) per anchor for the factorisation,
// so O(M^4 / 3) in all. The anchors are independent blocks; the paper's M <= 200 fits in registers.
//
// FP64 throughout.  Limits: M <= 256, lambda > 0 (the dual form), no shared increments.
#include <hip/hip_runtime.h>

#include <cmath>

#include "fbsde_host.hpp"
#include "fbsde_gram.hpp"
#include "fbsde_spd.hpp"

namespace {

using namespace fbsde;

constexpr int LMAX = 256;   // largest M of the register-resident factorisation

// Forward sweep (Algorithm 1, eq. Xk): W^j_N = sum_k sqrt(dt) xi^j_k for every point, particle and
// 4-coordinate group, accumulated in level order; the row pad up to ldw is written as zero.
// With all_levels the row of every level k = 0..N is stored, at W + k P M ldw (level 0 is zero).
__global__ void __launch_bounds__(256)
k_lit_forward(double* __restrict__ W, int64_t ldw, int M, int d, int N, double sqdt, uint32_t point_base,
              uint32_t k0, uint32_t k1, int64_t P, int all_levels) {
    const int ngl = (int)(ldw / 4);
    const int64_t n = P * (int64_t)M * ngl;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const int g = (int)(t % ngl);
        const int64_t pj = t / ngl;
        const int j = (int)(pj % M);
        const int64_t p = pj / M;
        double w[4] = {0.0, 0.0, 0.0, 0.0};
        double* row = W + pj * ldw + 4 * g;
        const int64_t lstride = P * (int64_t)M * ldw;
        if (all_levels) {
#pragma unroll
            for (int e = 0; e < 4; ++e) row[e] = 0.0;
        }
        for (int k = 0; k < N; ++k) {
            if (4 * g < d) {
                double z[4];
                increment4<double>((uint32_t)g, (uint32_t)j, (uint32_t)k, point_base + (uint32_t)p, k0, k1, z);
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] += sqdt * z[e];
            }
            if (all_levels) {
                double* rk = row + (int64_t)(k + 1) * lstride;
#pragma unroll
                for (int e = 0; e < 4; ++e) rk[e] = (4 * g + e < d) ? w[e] : 0.0;
            }
        }
        if (!all_levels) {
#pragma unroll
            for (int e = 0; e < 4; ++e) row[e] = (4 * g + e < d) ? w[e] : 0.0;
        }
    }
}

// Terminal condition Y^j_N = g(x0 + mu T + s W^j_N) (one wave per particle row).  Grid (M, P).
__global__ void __launch_bounds__(64)
k_lit_terminal(const double* __restrict__ W, int64_t ldw, int M, int d, const double* __restrict__ x0,
               const double* __restrict__ mu, const double* __restrict__ gvec, double s, double T, int g_kind,
               double ga, double gb, double* __restrict__ Y, uint32_t* __restrict__ status) {
    const int j = blockIdx.x, p = blockIdx.y;
    const double* row = W + ((int64_t)p * M + j) * ldw;
    const double* xp = x0 + (int64_t)p * d;
    const bool dot = g_dot_arg(g_kind);
    double q = 0.0;
    for (int i = threadIdx.x; i < d; i += 64) {
        const double X = xp[i] + (mu ? mu[i] * T : 0.0) + s * row[i];
        q += dot ? gvec[i] * X : X * X;
    }
    q = wave_sum(q);
    if (threadIdx.x == 0) {
        const double y = g_of(g_kind, ga, gb, q, d);
        Y[(int64_t)p * M + j] = y;
        if (!isfinite(y)) atomicOr(&status[p], (uint32_t)ST_NONFINITE);
    }
}

// W_k = W_{k+1} - sqrt(dt) xi_k for every point, particle and 4-coordinate group (zero: W_0 = 0).
__global__ void __launch_bounds__(256)
k_lit_reverse(double* __restrict__ W, int64_t ldw, int M, int d, int k, double sqdt, uint32_t point_base,
              uint32_t k0, uint32_t k1, int64_t P, int zero) {
    const int ng = (d + 3) / 4;
    const int64_t n = P * (int64_t)M * ng;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const int g = (int)(t % ng);
        const int64_t pj = t / ng;
        const int j = (int)(pj % M);
        const int64_t p = pj / M;
        double* row = W + pj * ldw + 4 * g;
        if (zero) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (4 * g + e < d) row[e] = 0.0;
            continue;
        }
        double z[4];
        increment4<double>((uint32_t)g, (uint32_t)j, (uint32_t)k, point_base + (uint32_t)p, k0, k1, z);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (4 * g + e < d) row[e] -= sqdt * z[e];
    }
}

// G = W W^T per point: 64 x 64 tiles of the lower triangle (mirrored on store), 4 x 4 outputs per
// thread, the coordinate axis staged through LDS 16 at a time.  The axis is split into `nsplit`
// chunks of `chunk` coordinates (a multiple of 16), one workgroup each, so that a launch has enough
// workgroups for the whole chip; chunk ks writes its partial matrix to Gpart[ks][P][M][M].
// Grid (tiles * nsplit, P).
__global__ void __launch_bounds__(256)
k_lit_gram(const double* __restrict__ W, int64_t ldw, int M, int ld, int ntiles, int chunk,
           double* __restrict__ Gpart) {
    __shared__ double As[64][17], Bs[64][17];
    const int ks = blockIdx.x / ntiles;
    int bi = 0, t = blockIdx.x % ntiles;
    while (t > bi) { t -= bi + 1; ++bi; }
    const int bj = t;
    const int p = blockIdx.y, tid = threadIdx.x;
    const int ty = tid / 16, tx = tid % 16;
    const double* Wp = W + (int64_t)p * M * ldw;
    const int r0 = 64 * bi, c0 = 64 * bj;
    double acc[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] = 0.0;
    const int kb = ks * chunk, ke = min(ld, kb + chunk);
    for (int k0 = kb; k0 < ke; k0 += 16) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = tid + 256 * q;
            const int row = e / 16, kk = e % 16;
            As[row][kk] = (r0 + row < M) ? Wp[(int64_t)(r0 + row) * ldw + k0 + kk] : 0.0;
            Bs[row][kk] = (c0 + row < M) ? Wp[(int64_t)(c0 + row) * ldw + k0 + kk] : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            double a[4], b[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) a[r] = As[4 * ty + r][kk];
#pragma unroll
            for (int c = 0; c < 4; ++c) b[c] = Bs[4 * tx + c][kk];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[r][c] += a[r] * b[c];
        }
        __syncthreads();
    }
    double* Gp = Gpart + ((int64_t)ks * gridDim.y + p) * M * M;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int i = r0 + 4 * ty + r, j = c0 + 4 * tx + c;
            if (i < M && j < M) {
                Gp[(int64_t)i * M + j] = acc[r][c];
                Gp[(int64_t)j * M + i] = acc[r][c];
            }
        }
}

// G = sum_ks Gpart[ks] over P M M elements and, with Rpart, rho = sum_ks Rpart[ks] over nr = P M
// elements, in chunk order (deterministic).  upper: Gpart holds the 16 x 16 tiles of the upper triangle only, which
// are mirrored (grid of whole matrices: element e = (p M + i) M + j).
__global__ void __launch_bounds__(256)
k_lit_gram_sum(const double* __restrict__ Gpart, const double* __restrict__ Rpart, int nsplit, int M, int upper,
               int64_t n, int64_t nr, double* __restrict__ G, double* __restrict__ rho) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        int64_t src = e;
        if (upper) {
            const int64_t row = e / M, p = row / M;
            const int i = (int)(row - p * M), j = (int)(e - row * M);
            if (i / 16 > j / 16) src = (p * M + j) * M + i;
        }
        double v = 0.0;
        for (int ks = 0; ks < nsplit; ++ks) v += Gpart[(int64_t)ks * n + src];
        G[e] = v;
        if (Rpart && e < nr) {
            double r = 0.0;
            for (int ks = 0; ks < nsplit; ++ks) r += Rpart[(int64_t)ks * nr + e];
            rho[e] = r;
        }
    }
}

// rho_j = sum_i W^j_i (one wave per particle row; the row pad is zero).  Grid (M, P).
__global__ void __launch_bounds__(64)
k_lit_rowsum(const double* __restrict__ W, int64_t ldw, int M, int ld, double* __restrict__ rho) {
    const int j = blockIdx.x, p = blockIdx.y;
    const double* row = W + ((int64_t)p * M + j) * ldw;
    double v = 0.0;
    for (int i = threadIdx.x; i < ld; i += 64) v += row[i];
    v = wave_sum(v);
    if (threadIdx.x == 0) rho[(int64_t)p * M + j] = v;
}

template <int NT>
__device__ __forceinline__ double block_sum(double v, double* red) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) s += red[w];
    __syncthreads();
    return s;
}

// One anchor m of point p at level k.  Grid (M, P), NW wavefronts.  The M x M dual system, bordered by its
// right-hand side, is built, factored and solved in registers as T x T tiles of the FP64 matrix cores
// (SpdSystem in fbsde_spd.hpp).  Bound by the chain of the elimination steps and by instruction issue, not by
// the matrix cores (64 points, per level, against an L D L^T in registers that broadcast one column a step
// through LDS: M = 20 26 -> 16 us, M = 50 74 -> 77 us, M = 64 0.21 -> 0.14 ms, M = 100 0.69 -> 0.39 ms, M = 128
// 1.8 -> 0.82 ms, M = 160 7.4 -> 1.8 ms, M = 200 11.2 -> 2.9 ms, M = 256 55 -> 9.3 ms).
//   eps2 = h^2 2 s^2 t_k d (0: uniform weights);  lam = ridge_rel s^2 t_{k+1} > 0.
template <int T>
__global__ void __launch_bounds__(64 * spd_waves(T), spd_occupancy(T))
k_lit_anchor(const double* __restrict__ G, int M, const double* __restrict__ rho, const double* __restrict__ Ynext,
             double* __restrict__ Ynew, double s, double dt, double eps2_all, const double* __restrict__ eps2_pp,
             double lam, FSpec f, int newton_iters, double* __restrict__ zstats, double* __restrict__ c_out,
             uint32_t* __restrict__ status) {
    constexpr int NW = spd_waves(T), NT = 64 * NW;
    __shared__ SpdShared<T> sh;
    __shared__ double2 og[16 * T];   // per particle: Om_i and G_im (zero beyond M)
    __shared__ double bv[16 * T];    // the responses, then the right-hand side Om Y
    __shared__ double red[NW];
    __shared__ double ybar_s;
    const int m = blockIdx.x, p = blockIdx.y, tid = threadIdx.x;
    const double* Gp = G + (int64_t)p * M * M;
    const double s2 = s * s;
    SpdSystem<T> sys;
    sys.init(blockIdx.x + gridDim.x * blockIdx.y);
    const double gmm = Gp[(int64_t)m * M + m];
    for (int j = tid; j < 16 * T; j += NT) {
        const bool in = j < M;
        const double gj = in ? Gp[(int64_t)m * M + j] : 0.0;
        og[j] = make_double2(0.0, gj);
        sh.x[j] = in ? s2 * (Gp[(int64_t)j * M + j] - 2.0 * gj + gmm) : 0.0;   // |D_j|^2, until the solve
        bv[j] = in ? Ynext[(int64_t)p * M + j] : 0.0;
    }
    __syncthreads();
    const double eps2 = eps2_pp ? eps2_pp[p] : eps2_all;
    // kernel weights of eq. Dj about the anchor (smallest squared distance subtracted) and the plain mean
    if (tid < 64) {
        double qmin = INFINITY, ys = 0.0;
        for (int j = tid; j < M; j += 64) {
            qmin = fmin(qmin, sh.x[j]);
            ys += bv[j];
        }
        qmin = wave_min(qmin);
        ys = wave_sum(ys);
        double es = 0.0;
        for (int j = tid; j < M; j += 64) {
            const double e = (eps2 > 0.0) ? exp(-(sh.x[j] - qmin) / eps2) : 1.0;
            og[j].x = e;
            es += e;
        }
        es = wave_sum(es);
        for (int j = tid; j < M; j += 64) {
            const double o = sqrt(og[j].x / es);
            og[j].x = o;
            bv[j] *= o;
        }
        if (tid == 0) ybar_s = ys / (double)M;
    }
    __syncthreads();

    // the system: Om (1 1^T + K) Om + lam I (Om is zero on the padding rows, which get a unit diagonal), and
    // the right-hand side in column np
    const int np = spd_pivots(M);
    auto load = [&](int i, int j) { return Gp[min(i, M - 1) * M + min(j, M - 1)]; };
    const bool good = sys.solve(
        load,
        [&](double Gij, int i, int j) {
            const double2 u = og[i], w = og[j];
            return u.x * w.x * fma(s2, Gij - u.y - w.y + gmm, 1.0);
        },
        [&](int i) { return (i < M) ? lam : 1.0; }, [&](int i) { return bv[i]; }, np, np, sh);
    uint32_t st = good ? 0u : (uint32_t)ST_NONFINITE;
    for (int j = tid; j < M; j += NT) sh.x[j] *= og[j].x;   // c = Om S^-1 Om Y
    __syncthreads();
    if (c_out) {   // x-dependent coefficients: Z needs alpha_x itself, formed by k_geo_alpha_z
        for (int j = tid; j < M; j += NT) c_out[((int64_t)p * M + m) * M + j] = sh.x[j];
        if ((tid & 63) == 0 && st) atomicOr(&status[p], st);
        return;
    }

    // c^T K c entry by entry (with the G_im terms taken out of the sum they cancel there: 1e-11 off instead of
    // 1e-15), and sum_j c_j (rho_j - rho_m)
    const double q = s2 * sys.quadratic([&](int i, int j) { return load(i, j) - og[i].y - og[j].y + gmm; }, sh);
    const double* rp = rho + (int64_t)p * M;
    const double rm = rp[m];
    double r = 0.0;
    for (int j = tid; j < M; j += NT) r += sh.x[j] * (rp[j] - rm);
    const double cKc = block_sum<NT>(q, red);
    const double crho = block_sum<NT>(r, red);
    if ((tid & 63) == 0) {
        if (tid == 0) {
            const double zz = s2 * cKc;          // |Z|^2, Z = s alpha_x
            const double zs = s2 * crho;         // sum_i Z_i
            double Fp;
            const double y = newton_y(f, ybar_s, zz, zs, dt, newton_iters, Fp, st);
            Ynew[(int64_t)p * M + m] = y;
            if (zstats) {
                zstats[((int64_t)p * M + m) * 2 + 0] = zz;
                zstats[((int64_t)p * M + m) * 2 + 1] = zs;
            }
        }
        if (st) atomicOr(&status[p], st);
    }
}

// ------------------------------------------------------------------ affine diagonal coefficient family
// mu(x) = mu0 x + mu1, sigma(x) = diag(sigma0 x + sigma1) (geometric: mu1 = sigma1 = 0).  The displacement
// V = X - x0 is stored at every level (the path cannot be reversed from its increments), V_k at
// Vs + k P M ldw.

// Forward sweep (eq. Xk): V_{k+1} = V_k + (mu0 X + mu1) dt + (sigma0 X + sigma1) sqrt(dt) xi_k with
// X = x0 + V_k, componentwise, V_0 = 0; one thread per (point, particle, 4-coordinate group), the row
// pad written as zero.
__global__ void __launch_bounds__(256)
k_geo_forward(double* __restrict__ Vs, int64_t ldw, int M, int d, int N, double dt, double sqdt, double mu0,
              double s0, double mu1, double s1, const double* __restrict__ x0, uint32_t point_base, uint32_t k0,
              uint32_t k1, int64_t P) {
    const int ngl = (int)(ldw / 4);
    const int64_t n = P * (int64_t)M * ngl;
    const int64_t lstride = P * (int64_t)M * ldw;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const int g = (int)(t % ngl);
        const int64_t pj = t / ngl;
        const int j = (int)(pj % M);
        const int64_t p = pj / M;
        double xg[4], v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 4; ++e) xg[e] = (4 * g + e < d) ? x0[p * d + 4 * g + e] : 0.0;
        double* row = Vs + pj * ldw + 4 * g;
#pragma unroll
        for (int e = 0; e < 4; ++e) row[e] = 0.0;
        for (int k = 0; k < N; ++k) {
            if (4 * g < d) {
                double z[4];
                increment4<double>((uint32_t)g, (uint32_t)j, (uint32_t)k, point_base + (uint32_t)p, k0, k1, z);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double X = xg[e] + v[e];
                    v[e] += (mu0 * X + mu1) * dt + (s0 * X + s1) * (sqdt * z[e]);
                }
            }
            double* rk = row + (int64_t)(k + 1) * lstride;
#pragma unroll
            for (int e = 0; e < 4; ++e) rk[e] = (4 * g + e < d) ? v[e] : 0.0;
        }
    }
}

// eps_k^2 = h2 2 (1/M) sum_j |V_j - Vbar|^2 = h2 2 (tr G / M - sum G / M^2) per point (one block each).
__global__ void __launch_bounds__(256)
k_geo_bandwidth(const double* __restrict__ G, int M, double h2, double* __restrict__ eps2) {
    __shared__ double red[4];
    const int p = blockIdx.x;
    const double* Gp = G + (int64_t)p * M * M;
    double tr = 0.0, tot = 0.0;
    for (int64_t e = threadIdx.x; e < (int64_t)M * M; e += 256) {
        const double g = Gp[e];
        tot += g;
        if (e / M == e % M) tr += g;
    }
    tr = block_sum<256>(tr, red);
    tot = block_sum<256>(tot, red);
    if (threadIdx.x == 0) eps2[p] = fmax(0.0, h2 * 2.0 * (tr / M - tot / ((double)M * M)));
}

// One level's slopes and Z of every anchor of the geometric family, from the dual solutions c of
// k_lit_anchor (c_out mode): alpha_x = sum_j c_j (V_j - V_m), the [M x M] . [M x d] product per point.
// One workgroup per (32-coordinate slice, point) holds the slice of all M displacements in LDS and serves
// every anchor from it.  Thread (g, i) = (tid / 32, tid % 32) takes
// coordinate i of the slice for the anchors m = g, g + 8, ...: alpha_i = sum_j c_mj V_ji - (sum_j c_mj) V_mi,
// Z_i = (sigma0 (x0_i + V_mi) + sigma1) alpha_i.  The slice's sums of Z_i^2 and Z_i per anchor go to
// part[(p M + m) nsl + slice][2] (reduced over the 32 lanes of a half wave).  Grid (nsl, P).
__global__ void __launch_bounds__(256)
k_geo_alpha_z(const double* __restrict__ Vk, int64_t ldw, int M, int d, const double* __restrict__ x0,
              const double* __restrict__ C, double s0, double s1, int nsl, double* __restrict__ part) {
    extern __shared__ double Vsl[];   // [M][33]
    const int sl = blockIdx.x, p = blockIdx.y, tid = threadIdx.x;
    const int i = tid & 31, g = tid >> 5;
    const int c0 = 32 * sl;
    const double* Vp = Vk + (int64_t)p * M * ldw;
    for (int e = tid; e < M * 32; e += 256) {
        const int j = e / 32, ii = e % 32;
        Vsl[j * 33 + ii] = (c0 + ii < d) ? Vp[(int64_t)j * ldw + c0 + ii] : 0.0;
    }
    __syncthreads();
    const bool in = c0 + i < d;
    const double xi = in ? x0[(int64_t)p * d + c0 + i] : 0.0;
    for (int m = g; m < M; m += 8) {
        const double* cm = C + ((int64_t)p * M + m) * M;
        double a = 0.0, cs = 0.0;
        for (int j = 0; j < M; ++j) {
            const double c = cm[j];
            a += c * Vsl[j * 33 + i];
            cs += c;
        }
        const double vm = Vsl[m * 33 + i];
        a -= cs * vm;
        const double z = in ? (s0 * (xi + vm) + s1) * a : 0.0;
        double zz = z * z, zs = z;
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) {   // within the 32 lanes of this anchor group
            zz += __shfl_xor(zz, off, 64);
            zs += __shfl_xor(zs, off, 64);
        }
        if (i == 0) {
            double* q = part + (((int64_t)p * M + m) * nsl + sl) * 2;
            q[0] = zz;
            q[1] = zs;
        }
    }
}

// Sums the slices' partials of one anchor in slice order, then Newton (eq. NRiter) from the plain mean.
// Grid (M, P), one wave.
__global__ void __launch_bounds__(64)
k_geo_newton(const double* __restrict__ part, int nsl, int M, const double* __restrict__ Ynext,
             double* __restrict__ Ynew, double dt, FSpec f, int newton_iters, double* __restrict__ zstats,
             uint32_t* __restrict__ status) {
    const int m = blockIdx.x, p = blockIdx.y, lane = threadIdx.x;
    double ys = 0.0;
    for (int j = lane; j < M; j += 64) ys += Ynext[(int64_t)p * M + j];
    ys = wave_sum(ys);
    if (lane == 0) {
        const double* q = part + ((int64_t)p * M + m) * nsl * 2;
        double zz = 0.0, zs = 0.0;
        for (int sl = 0; sl < nsl; ++sl) {
            zz += q[2 * sl];
            zs += q[2 * sl + 1];
        }
        uint32_t st = 0;
        double Fp;
        const double y = newton_y(f, ys / (double)M, zz, zs, dt, newton_iters, Fp, st);
        Ynew[(int64_t)p * M + m] = y;
        if (zstats) {
            zstats[((int64_t)p * M + m) * 2 + 0] = zz;
            zstats[((int64_t)p * M + m) * 2 + 1] = zs;
        }
        if (st) atomicOr(&status[p], st);
    }
}

// u_p = mean_m Y^m (one wave per point).
__global__ void __launch_bounds__(64) k_lit_mean(const double* __restrict__ Y, int M, double* __restrict__ u) {
    const int p = blockIdx.x;
    double v = 0.0;
    for (int j = threadIdx.x; j < M; j += 64) v += Y[(int64_t)p * M + j];
    v = wave_sum(v);
    if (threadIdx.x == 0) u[p] = v / (double)M;
}

struct LitWS {
    double *W, *Ya, *Yb, *G, *rho, *Gpart, *Rpart, *C, *eps2, *Zpart;
};

// Coefficient family of a literal solve: sigma = s I with constant drift (geo = false), or the affine
// diagonal family mu(x) = mu0 x + mu1, sigma(x) = diag(sigma0 x + sigma1) (geometric: mu1 = sigma1 = 0).
struct Coef {
    bool geo;
    double mu0, s0, mu1, s1;
};

// Split of the Gram contraction.  M <= 128: k_gram, the whole triangle in one block, which a compute unit holds one
// of: about two a unit; otherwise 64 x 64 tiles of the lower triangle, about 2048 workgroups.  At least 256
// coordinates per workgroup either way.
struct GramSplit {
    bool rows;
    int ntiles, nsplit, chunk;
};
GramSplit gram_split(int64_t P, int64_t M, int64_t ld) {
    GramSplit g;
    g.rows = M <= 128;
    const int nb = (int)((M + 63) / 64);
    g.ntiles = g.rows ? 1 : nb * (nb + 1) / 2;
    const int64_t tp = g.ntiles * std::max<int64_t>(P, 1);   // P = 0: a size query with nothing to split
    const int64_t want = ((g.rows ? 512 : 2048) + tp - 1) / tp;
    g.nsplit = (int)std::max<int64_t>(1, std::min<int64_t>(want, ld / 256));
    g.chunk = (int)host::round_up((ld + g.nsplit - 1) / g.nsplit, g.rows ? GRAM_SLICE : 16);
    return g;
}

// Workspace: the state (scalar family: W_k, one level, reversed in place; geometric family: V_k for
// k = 0..N), two Y buffers, the Gram matrices and row sums with their per-chunk partials, and for the
// geometric family the dual solutions C [P][M][M] and the per-point bandwidths.
size_t lit_carve(int64_t P, int64_t M, int64_t N, int64_t ld, bool geo, char* base, LitWS& w, bool stored = false) {
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* ptr = base ? base + off : nullptr;
        off += (bytes + 255) / 256 * 256;
        return (double*)ptr;
    };
    w.W = take((size_t)((geo || stored) ? N + 1 : 1) * P * M * ld * 8);
    w.Ya = take((size_t)P * M * 8);
    w.Yb = take((size_t)P * M * 8);
    w.G = take((size_t)P * M * M * 8);
    w.rho = take((size_t)P * M * 8);
    const GramSplit gs = gram_split(P, M, ld);
    w.Gpart = (gs.nsplit > 1) ? take((size_t)gs.nsplit * P * M * M * 8) : w.G;
    // row sums: fused into the row-resident Gram kernel (partials per chunk), else their own kernel
    w.Rpart = !gs.rows ? nullptr : (gs.nsplit > 1) ? take((size_t)gs.nsplit * P * M * 8) : w.rho;
    w.C = geo ? take((size_t)P * M * M * 8) : nullptr;
    w.eps2 = geo ? take((size_t)P * 8) : nullptr;
    w.Zpart = geo ? take((size_t)P * M * ((ld + 31) / 32) * 2 * 8) : nullptr;   // per 32-coordinate slice
    return off;
}

int lit_check(const fbsde_problem* pb, int64_t P, host::Plan& pl) {
    int rc = host::check_problem(pb, P);
    if (rc) return rc;
    if (pb->prec != FBSDE_F64 || pb->shared_dw != 0 || host::per_point_forward_only(pb)) return FBSDE_EINVAL;
    if (pb->M > LMAX || !(pb->ridge_rel > 0.0)) return FBSDE_EINVAL;
    return host::make_plan(pb, P, pl);
}

int coef_check(const fbsde_problem* pb, const fbsde_coef* coef, Coef& c) {
    if (!coef || coef->reserved != 0) return FBSDE_EINVAL;
    if (coef->kind != FBSDE_COEF_GEOMETRIC && coef->kind != FBSDE_COEF_AFFINE_DIAG) return FBSDE_EINVAL;
    if (coef->kind == FBSDE_COEF_GEOMETRIC && (coef->mu1 != 0.0 || coef->sigma1 != 0.0)) return FBSDE_EINVAL;
    const double v[4] = {coef->mu0, coef->sigma0, coef->mu1, coef->sigma1};
    for (double x : v)
        if (!std::isfinite(x)) return FBSDE_EINVAL;
    if (!(coef->sigma0 * coef->sigma0 + coef->sigma1 * coef->sigma1 > 0.0)) return FBSDE_EINVAL;
    if (pb && pb->mu) return FBSDE_EINVAL;   // the family's drift replaces the constant one
    c = {true, coef->mu0, coef->sigma0, coef->mu1, coef->sigma1};
    return FBSDE_OK;
}

int anchors(int64_t P, int M, const double* G, const double* rho, const double* Yn, double* Y, double s, double dt,
            double eps2, double lam, FSpec f, int it, double* zst, uint32_t* status, hipStream_t st,
            const double* eps2_pp, double* c_out) {
    if (M > LMAX) return FBSDE_EINVAL;
#define LIT_ANCHOR(T)                                                                                               \
    case T:                                                                                                          \
        hipLaunchKernelGGL((k_lit_anchor<T>), dim3(M, (unsigned)P), dim3(64 * spd_waves(T)), 0, st, G, M, rho, Yn, Y, \
                           s, dt, eps2, eps2_pp, lam, f, it, zst, c_out, status);                                    \
        return FBSDE_OK;
    switch (spd_tiles(M)) {
        LIT_ANCHOR(1) LIT_ANCHOR(2) LIT_ANCHOR(3) LIT_ANCHOR(4) LIT_ANCHOR(5) LIT_ANCHOR(6) LIT_ANCHOR(7) LIT_ANCHOR(8)
        LIT_ANCHOR(9) LIT_ANCHOR(10) LIT_ANCHOR(11) LIT_ANCHOR(12) LIT_ANCHOR(13) LIT_ANCHOR(14) LIT_ANCHOR(15)
        LIT_ANCHOR(16) LIT_ANCHOR(17)
        default: return FBSDE_EINVAL;
    }
#undef LIT_ANCHOR
}

// The whole literal solve for either coefficient family (arguments validated by the callers).
void gram_rows(int64_t P, int M, const double* X, int ld, const GramSplit& gs, const LitWS& w, hipStream_t st) {
    switch ((M + 15) / 16) {
#define LIT_GRAM(NT)                                                                                                   \
    case NT:                                                                                                           \
        hipLaunchKernelGGL((k_gram<double, NT, GRAM_PLAIN>), dim3(gs.nsplit, (unsigned)P), dim3(256), 0, st, X,        \
                           (int64_t)ld, M, ld, M, gs.chunk, 1.0, nullptr, nullptr, w.Gpart, w.Rpart);                     \
        break;
        LIT_GRAM(1) LIT_GRAM(2) LIT_GRAM(3) LIT_GRAM(4) LIT_GRAM(5) LIT_GRAM(6) LIT_GRAM(7) LIT_GRAM(8)
#undef LIT_GRAM
    }
}

int lit_run(const fbsde_problem* pb, const Coef& cf, const host::Plan& pl, int64_t P, int32_t k_stop,
            const double* x0, double* u, double* Y_out, double* z_stats, uint32_t* status, const LitWS& w,
            hipStream_t st, bool stored = false) {
    int rc = FBSDE_OK;
    const int M = (int)pb->M, d = (int)pb->d;
    const host::Keys ky = host::keys_of(pb);
    const double dt = pb->T / (double)pb->N, sqdt = std::sqrt(dt);
    // the regression is in X-space: the scalar family's state is W (X = x0 + mu t + s W), the geometric
    // family's is V = X - x0
    const double s = cf.geo ? 1.0 : pb->s;
    const int64_t lstride = P * (int64_t)M * pl.ld;
    // forward sweep over every (point, particle, 4-coordinate group) and the terminal condition
    host::clear_status(status, P, st);
    const int64_t nfwd = P * (int64_t)M * (pl.ld / 4);
    const unsigned fblocks = (unsigned)std::min<int64_t>((nfwd + 255) / 256, (int64_t)1 << 20);
    if (cf.geo) {
        hipLaunchKernelGGL(k_geo_forward, dim3(fblocks), dim3(256), 0, st, w.W, (int64_t)pl.ld, M, d, (int)pb->N, dt,
                           sqdt, cf.mu0, cf.s0, cf.mu1, cf.s1, x0, pb->point_base, ky.k0, ky.k1, P);
        hipLaunchKernelGGL(k_lit_terminal, dim3(M, (unsigned)P), dim3(64), 0, st, w.W + pb->N * lstride,
                           (int64_t)pl.ld, M, d, x0, nullptr, pb->gvec, 1.0, pb->T, pb->g_kind, pb->gp[0], pb->gp[1],
                           w.Ya, status);
    } else {
        hipLaunchKernelGGL(k_lit_forward, dim3(fblocks), dim3(256), 0, st, w.W, (int64_t)pl.ld, M, d, (int)pb->N, sqdt,
                           pb->point_base, ky.k0, ky.k1, P, stored ? 1 : 0);
        hipLaunchKernelGGL(k_lit_terminal, dim3(M, (unsigned)P), dim3(64), 0, st, stored ? w.W + pb->N * lstride : w.W,
                           (int64_t)pl.ld, M, d, x0, pb->mu, pb->gvec, s, pb->T, pb->g_kind, pb->gp[0], pb->gp[1], w.Ya,
                           status);
    }
    const GramSplit gs = gram_split(P, M, pl.ld);
    const int64_t nG = P * (int64_t)M * M;
    const unsigned sblocks = (unsigned)std::min<int64_t>((nG + 255) / 256, (int64_t)1 << 16);
    const double gram_flops = (double)P * M * (M + 1.0) * d;
    const double anchor_flops = (double)P * M * (2.0 / 3.0 * std::pow(M + 1.0, 3) + 6.0 * M * (double)M);
    const int64_t ngroups = P * (int64_t)M * ((d + 3) / 4);
    const unsigned rblocks = (unsigned)std::min<int64_t>((ngroups + 255) / 256, (int64_t)1 << 20);
    const FSpec f = host::fspec_of(pb);
    // lambda_k = ridge_rel sigma^2 t_{k+1}, sigma^2 = sigma0^2 + sigma1^2 for the affine diagonal family
    const double s_ridge = cf.geo ? std::sqrt(cf.s0 * cf.s0 + cf.s1 * cf.s1) : pb->s;
    double* Yn = w.Ya;
    double* Yk = w.Yb;
    for (int k = (int)pb->N - 1; k >= k_stop; --k) {
        double* Xk = w.W;
        if (cf.geo || stored) Xk = w.W + k * lstride;
        else
            hipLaunchKernelGGL(k_lit_reverse, dim3(rblocks), dim3(256), 0, st, w.W, (int64_t)pl.ld, M, d, k, sqdt,
                               pb->point_base, ky.k0, ky.k1, P, k == 0 ? 1 : 0);
        const long tg = host::timer_begin(st, gram_flops, FBSDE_TIMED_LITERAL_GRAM);
        if (gs.rows) gram_rows(P, M, Xk, pl.ld, gs, w, st);
        else
            hipLaunchKernelGGL(k_lit_gram, dim3(gs.ntiles * gs.nsplit, (unsigned)P), dim3(256), 0, st, Xk,
                               (int64_t)pl.ld, M, pl.ld, gs.ntiles, gs.chunk, w.Gpart);
        if (gs.nsplit > 1)
            hipLaunchKernelGGL(k_lit_gram_sum, dim3(sblocks), dim3(256), 0, st, w.Gpart, gs.rows ? w.Rpart : nullptr,
                               gs.nsplit, M, gs.rows ? 1 : 0, nG, P * (int64_t)M, w.G, w.rho);
        host::timer_end(tg, st);
        if (!gs.rows && !cf.geo)
            hipLaunchKernelGGL(k_lit_rowsum, dim3(M, (unsigned)P), dim3(64), 0, st, Xk, (int64_t)pl.ld, M, pl.ld,
                               w.rho);
        double eps2 = 0.0;
        if (cf.geo)
            hipLaunchKernelGGL(k_geo_bandwidth, dim3((unsigned)P), dim3(256), 0, st, w.G, M,
                               k == 0 ? 0.0 : pb->eps_h * pb->eps_h, w.eps2);
        else if (pb->eps_h != 0.0 && k != 0)
            eps2 = pb->eps_h * pb->eps_h * 2.0 * s * s * (k * dt) * d;
        const double lam = pb->ridge_rel * s_ridge * s_ridge * ((k + 1) * dt);
        double* zst = (k == k_stop) ? z_stats : nullptr;
        const long ta = host::timer_begin(st, anchor_flops, FBSDE_TIMED_LITERAL_ANCHORS);
        rc = anchors(P, M, w.G, w.rho, Yn, Yk, s, dt, eps2, lam, f, pb->newton_iters, zst, status, st,
                     cf.geo ? w.eps2 : nullptr, cf.geo ? w.C : nullptr);
        host::timer_end(ta, st);
        if (rc) return rc;
        if (cf.geo) {
            const int nsl = (d + 31) / 32;
            const size_t lds = (size_t)M * 33 * 8;
            if (lds > 65536 &&
                hipFuncSetAttribute((const void*)k_geo_alpha_z, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
                    hipSuccess)
                return FBSDE_EHIP;
            hipLaunchKernelGGL(k_geo_alpha_z, dim3(nsl, (unsigned)P), dim3(256), lds, st, Xk,
                               (int64_t)pl.ld, M, d, x0, w.C, cf.s0, cf.s1, nsl, w.Zpart);
            hipLaunchKernelGGL(k_geo_newton, dim3(M, (unsigned)P), dim3(64), 0, st, w.Zpart, nsl, M, Yn, Yk, dt, f,
                               pb->newton_iters, zst, status);
        }
        std::swap(Yn, Yk);
    }
    hipLaunchKernelGGL(k_lit_mean, dim3((unsigned)P), dim3(64), 0, st, Yn, M, u);
    if (Y_out) (void)hipMemcpyAsync(Y_out, Yn, (size_t)P * M * 8, hipMemcpyDeviceToDevice, st);
    return host::last_error();
}

}  // namespace

extern "C" {

int fbsde_literal_workspace_size(const fbsde_problem* pb, int64_t P, size_t* bytes) {
    if (!bytes) return FBSDE_EINVAL;
    host::Plan pl;
    const int rc = lit_check(pb, P, pl);
    if (rc) return rc;
    LitWS w;
    *bytes = lit_carve(P, pb->M, pb->N, pl.ld, false, nullptr, w);
    return FBSDE_OK;
}

int fbsde_literal_workspace_size_stored(const fbsde_problem* pb, int64_t P, size_t* bytes) {
    if (!bytes) return FBSDE_EINVAL;
    host::Plan pl;
    const int rc = lit_check(pb, P, pl);
    if (rc) return rc;
    LitWS w;
    *bytes = lit_carve(P, pb->M, pb->N, pl.ld, false, nullptr, w, true);
    return FBSDE_OK;
}

int fbsde_solve_literal(const fbsde_problem* pb, int64_t P, int32_t k_stop, const double* x0, double* u,
                        double* Y_out, double* z_stats, uint32_t* status, void* wsp, size_t ws_bytes,
                        fbsde_stream stream) {
    host::Plan pl;
    int rc = lit_check(pb, P, pl);
    if (rc) return rc;
    if (k_stop < 0 || k_stop >= pb->N) return FBSDE_EINVAL;
    if (P == 0) return FBSDE_OK;   // nothing is read or written; the pointers may be null
    if (!x0 || !u || !status || !wsp) return FBSDE_EINVAL;
    LitWS w;
    // a workspace that holds every level selects the stored path (no reversal by regenerated increments)
    const bool stored = lit_carve(P, pb->M, pb->N, pl.ld, false, nullptr, w, true) <= ws_bytes;
    if (!stored && lit_carve(P, pb->M, pb->N, pl.ld, false, nullptr, w) > ws_bytes) return FBSDE_ENOSPC;
    lit_carve(P, pb->M, pb->N, pl.ld, false, (char*)wsp, w, stored);
    return lit_run(pb, Coef{false, 0.0, 0.0, 0.0, 0.0}, pl, P, k_stop, x0, u, Y_out, z_stats, status, w,
                   (hipStream_t)stream, stored);
}

int fbsde_literal_coef_workspace_size(const fbsde_problem* pb, const fbsde_coef* coef, int64_t P, size_t* bytes) {
    if (!bytes) return FBSDE_EINVAL;
    host::Plan pl;
    int rc = lit_check(pb, P, pl);
    if (rc) return rc;
    Coef cf;
    if ((rc = coef_check(pb, coef, cf))) return rc;
    LitWS w;
    *bytes = lit_carve(P, pb->M, pb->N, pl.ld, true, nullptr, w);
    return FBSDE_OK;
}

int fbsde_solve_literal_coef(const fbsde_problem* pb, const fbsde_coef* coef, int64_t P, int32_t k_stop,
                             const double* x0, double* u, double* Y_out, double* z_stats, uint32_t* status, void* wsp,
                             size_t ws_bytes, fbsde_stream stream) {
    host::Plan pl;
    int rc = lit_check(pb, P, pl);
    if (rc) return rc;
    Coef cf;
    if ((rc = coef_check(pb, coef, cf))) return rc;
    if (k_stop < 0 || k_stop >= pb->N) return FBSDE_EINVAL;
    if (P == 0) return FBSDE_OK;   // nothing is read or written; the pointers may be null
    if (!x0 || !u || !status || !wsp) return FBSDE_EINVAL;
    LitWS w;
    if (lit_carve(P, pb->M, pb->N, pl.ld, true, nullptr, w) > ws_bytes) return FBSDE_ENOSPC;
    lit_carve(P, pb->M, pb->N, pl.ld, true, (char*)wsp, w);
    return lit_run(pb, cf, pl, P, k_stop, x0, u, Y_out, z_stats, status, w, (hipStream_t)stream);
}

}  // extern "C"
