// Gram matrices of at most 128 rows or columns on the FP64 matrix cores (16 x 16 x 4 products), for the direct
// level solves (fbsde_direct.hpp) and the literal scheme (fbsde_literal.hip).
//
// Two waves share a contiguous part of the contraction, 8 or 16 indices a step, and hold half of the 16 x 16 tiles
// of the upper triangle each (NT tiles per side: 18 at most, 144 of a lane's 256 registers; with the whole triangle
// in one wave the compiler copies the tiles between its two register files every step).  Lane l holds row l % 16 of
// an operand tile at contraction index l / 16, for the left and the right operand alike, so one register serves tile
// row i and tile column j: NT operand registers feed up to 18 independent products, straight from memory, without LDS
// and without a barrier, and the next step's loads have a whole step to arrive.  The block's two parts are summed
// through LDS at the end, in order.
// Bound by the matrix cores.  Against operands staged through LDS for a block-wide tiling with two barriers a step
// (direct solve) and register blocks on the vector units (literal scheme), per level:
// literal scheme, 64 points, M = 100, d = 10^4 343 -> 174 us (53 TFLOP/s over the tiles); direct primal, 512 points,
// M = 1024, d = 100 235 -> 141 us (53 TFLOP/s); direct dual, 64 points, M = 100, d = 500 22 -> 17 us and d = 100 15 -> 13;
// one point, M = 512, d = 100 10 -> 7 us.
#pragma once
#include "fbsde_rowteam.hpp"
#include "fbsde_spd.hpp"

namespace fbsde {

constexpr int gram_ntile(int nt) { return nt * (nt + 1) / 2; }
// The 16 x 16 tiles of an n x n matrix's upper triangle, row by row, without the padding beyond n: the rows of tile
// row t one after the other, n - 16 t entries each.  At most n^2 entries (whole tiles are 6 kB at n = 17, the square 2.3).
__host__ __device__ constexpr int gram_row(int n, int t) { return 16 * t * n - 128 * t * (t - 1); }   // where tile row t begins
__host__ __device__ constexpr int gram_entries(int n) { return gram_row(n, n / 16) + (n % 16) * (n - n / 16 * 16); }
__device__ __forceinline__ int gram_index(int n, int i, int j) {   // j's tile not left of i's
    const int t = i >> 4;
    return gram_row(n, t) + (i & 15) * (n - 16 * t) + j - 16 * t;
}
constexpr int GRAM_SLICE = 32;   // a block's slice of the contraction is a multiple of this: 16 indices a part

// What is multiplied:
//   GRAM_DUAL    f_i f_j sum_c (W_ic - Wbar_c) (W_jc - Wbar_c), f = s w^1/2: rows of the cloud, contracted over the
//                coordinates (ld, a multiple of 16);
//   GRAM_PRIMAL  s^2 sum_j w_j (W_ja - Wbar_a) (W_jb - Wbar_b): columns, contracted over the particles;
//   GRAM_PLAIN   sum_c W_ic W_jc, and the row sums sum_c W_ic.
enum { GRAM_DUAL = 0, GRAM_PRIMAL = 1, GRAM_PLAIN = 2 };

// n = 2 or 4 neighbouring elements
template <int n>
__device__ __forceinline__ void gram_load(const double* p, double v[n]) {
#pragma unroll
    for (int e = 0; e < n; e += 2) {
        const double2 a = *reinterpret_cast<const double2*>(p + e);
        v[e] = a.x; v[e + 1] = a.y;
    }
}
template <int n>
__device__ __forceinline__ void gram_load(const float* p, float v[n]) {
#pragma unroll
    for (int e = 0; e < n; e += 2) {
        const float2 a = *reinterpret_cast<const float2*>(p + e);
        v[e] = a.x; v[e + 1] = a.y;
    }
}

// The products of one wave: tiles T0 <= q < T1 of the triangle (by rows) over the indices k0 <= k < k1, and for
// GRAM_PLAIN the lane's share of its rows' sums.  Rows past the last are the last one again: multiplied by a zero
// factor or weight by what follows, or not written.
template <typename S, int NT, int KIND, int T0, int T1>
__device__ __forceinline__ void gram_part(const S* __restrict__ Wp, int64_t ldw, int M, int k0, int k1, double s2,
                                          const double* __restrict__ wb, const double* __restrict__ wp, int g, int c,
                                          spd_v4 (&acc)[T1 > T0 ? T1 - T0 : 1], double (&rsl)[NT]) {
    constexpr bool PRIMAL = KIND == GRAM_PRIMAL;
    constexpr int KE = (NT > 4) ? 2 : 4;   // contraction indices a lane takes a step
    const S* row[PRIMAL ? 1 : NT];
    double wbc[NT];
    if constexpr (PRIMAL) {
        row[0] = Wp + c;
#pragma unroll
        for (int i = 0; i < NT; ++i) wbc[i] = wb[16 * i + c];
    } else {
#pragma unroll
        for (int i = 0; i < NT; ++i) row[i] = Wp + (int64_t)min(16 * i + c, M - 1) * ldw + KE * g;
    }
    S nx[NT][KE];
    double nw[KE];   // PRIMAL: the weights of the step's particles; DUAL: the mean of its coordinates
    auto fetch = [&](int kc) {
        if constexpr (PRIMAL) {
#pragma unroll
            for (int e = 0; e < KE; ++e) {
                const int j = kc + 4 * e + g;
                const S* r = row[0] + (int64_t)min(j, M - 1) * ldw;
#pragma unroll
                for (int i = 0; i < NT; ++i) nx[i][e] = r[16 * i];
                nw[e] = wp[min(j, M - 1)];
            }
        } else {
#pragma unroll
            for (int i = 0; i < NT; ++i) gram_load<KE>(row[i] + kc, nx[i]);
            if constexpr (KIND == GRAM_DUAL) gram_load<KE>(wb + kc + KE * g, nw);
        }
    };
    const int last = k0 + (k1 - k0 - 1) / (4 * KE) * (4 * KE);
    fetch(k0);
    for (int kc = k0; kc < k1; kc += 4 * KE) {
        double x[NT][KE], wk[KE];
#pragma unroll
        for (int e = 0; e < KE; ++e) {
            // the weight past the slice's end is dropped here and not where it is fetched: used at once, its load keeps
            // the step's other loads behind it (256 -> 370 us, 8 points, M = 10^5, d = 128)
            wk[e] = (PRIMAL && kc + 4 * e + g >= k1) ? 0.0 : nw[e];
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                if constexpr (PRIMAL) x[i][e] = (double)nx[i][e] - wbc[i];
                else if constexpr (KIND == GRAM_DUAL) x[i][e] = (double)nx[i][e] - wk[e];
                else {
                    x[i][e] = (double)nx[i][e];
                    if (T0 == 0) rsl[i] += x[i][e];
                }
            }
        }
        fetch(min(kc + 4 * KE, last));   // at the end the last step again: no branch splits the loop's body
        asm volatile("" ::: "memory");   // the loads stay above the products
#pragma unroll
        for (int e = 0; e < KE; ++e) {
            double y[NT];
            const double sw = PRIMAL ? s2 * wk[e] : 1.0;
#pragma unroll
            for (int j = 0; j < NT; ++j) y[j] = PRIMAL ? sw * x[j][e] : x[j][e];
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = i; j < NT; ++j) {
                    const int q = i * NT - i * (i - 1) / 2 + j - i;
                    if (q >= T0 && q < T1)
                        acc[q - T0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i][e], y[j], acc[q - T0], 0, 0, 0);
                }
        }
    }
}

// Grid (slices, P).  out: DUAL and PRIMAL [P][slices][gram_entries(n)] (n = M, d), PLAIN [slices][P][M][M], the upper
// triangle's tiles only unless there is but one slice, and rsum [slices][P][M].
template <typename S, int NT, int KIND>
__global__ void __launch_bounds__(256, 2)
k_gram(const S* __restrict__ W, int64_t ldw, int M, int ld, int n, int slice, double s, const double* __restrict__ Wbar,
       const double* __restrict__ w, double* __restrict__ out, double* __restrict__ rsum) {
    constexpr int NTILE = gram_ntile(NT), TH = NTILE / 2, TM = NTILE - TH;
    constexpr int CH = TM < 6 ? TM : 6;   // tiles of each half a round of the reduction takes
    __shared__ double red[2][2 * CH][256];
    __shared__ double rs2[2][16 * NT];
    __shared__ double f[16 * NT];
    const int p = blockIdx.y, t = threadIdx.x, lane = t & 63, g = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), half = wave & 1, part = wave >> 1;
    const S* Wp = W + (int64_t)p * M * ldw;
    const double* wb = Wbar + (int64_t)p * ld;
    const double* wp = w + (int64_t)p * M;
    const int len = (KIND == GRAM_PRIMAL) ? M : ld;
    const int b0 = blockIdx.x * slice, b1 = min(b0 + slice, len);
    const int sub = ((b1 - b0 + 1) / 2 + 15) / 16 * 16;
    const int k0 = b0 + part * sub, k1 = min(k0 + sub, b1);
    if constexpr (KIND == GRAM_DUAL) {
        if (t < 16 * NT) f[t] = (t < M) ? s * sqrt(wp[t]) : 0.0;
    }
    spd_v4 acc[TM];
#pragma unroll
    for (int q = 0; q < TM; ++q) acc[q] = spd_v4{0.0, 0.0, 0.0, 0.0};
    double rsl[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) rsl[i] = 0.0;
    if (k0 < k1) {
        if (half) gram_part<S, NT, KIND, 0, TM>(Wp, ldw, M, k0, k1, s * s, wb, wp, g, c, acc, rsl);
        else if constexpr (TH > 0) {
            spd_v4 low[TH];
#pragma unroll
            for (int q = 0; q < TH; ++q) low[q] = acc[q];
            gram_part<S, NT, KIND, TM, NTILE>(Wp, ldw, M, k0, k1, s * s, wb, wp, g, c, low, rsl);
#pragma unroll
            for (int q = 0; q < TH; ++q) acc[q] = low[q];
        }
    }
    if constexpr (KIND == GRAM_PLAIN) {
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            rsl[i] += __shfl_xor(rsl[i], 16, 64);
            rsl[i] += __shfl_xor(rsl[i], 32, 64);
            if (half && g == 0) rs2[part][16 * i + c] = rsl[i];
        }
    }
    double* po = (KIND == GRAM_PLAIN) ? out + ((int64_t)blockIdx.x * gridDim.y + p) * M * M
                                      : out + ((int64_t)p * gridDim.x + blockIdx.x) * gram_entries(n);
#pragma unroll
    for (int q0 = 0; q0 < TM; q0 += CH) {
        if (q0) __syncthreads();   // the tiles before have been read
#pragma unroll
        for (int q = q0; q < q0 + CH; ++q)
            if (q < TM) {
#pragma unroll
                for (int r = 0; r < 4; ++r) red[part][(half ? 0 : CH) + q - q0][64 * r + lane] = acc[q < TM ? q : 0][r];
            }
        __syncthreads();
        if (q0 == 0 && KIND == GRAM_PLAIN) {
            if (t < M) rsum[((int64_t)blockIdx.x * gridDim.y + p) * M + t] = rs2[0][t] + rs2[1][t];
        }
        auto put = [&](int q, int slot) {   // tile q, element t
            const double v = red[0][slot][t] + red[1][slot][t];
            int ti = 0, tj = q;
            while (tj >= NT) { ++ti; tj += ti - NT; }
            const int i = 16 * ti + (t >> 4), j = 16 * tj + (t & 15);
            if (tj == NT - 1 && (i >= n || j >= n)) return;   // padding, in the last tile column only
            if constexpr (KIND == GRAM_PRIMAL) po[gram_index(n, i, j)] = v;
            else if constexpr (KIND == GRAM_DUAL) po[gram_index(n, i, j)] = f[i] * f[j] * v;
            else {
                po[(int64_t)i * n + j] = v;
                if (gridDim.x == 1 && ti != tj) po[(int64_t)j * n + i] = v;   // no sum over slices follows
            }
        };
#pragma unroll
        for (int q = q0; q < q0 + CH; ++q) {
            if (q < TM) put(q, q - q0);
            if (q < TH) put(TM + q, CH + q - q0);
        }
    }
}

}  // namespace fbsde
