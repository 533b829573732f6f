// Symmetric positive definite systems of up to 256 unknowns, one block each, factored and solved in
// registers on the FP64 matrix cores.  Used for the M x M systems of the paper-literal anchors and for the
// per-point ridge systems that are solved directly.
//
// Layout.  The upper triangle of the matrix, bordered by the right-hand side as an extra column, is cut into
// 16 x 16 tiles (i, j), i <= j < T.  Wave 0 owns the diagonal tiles, the other NW - 1 waves share the rest row
// by row.  A tile is one accumulator of v_mfma_f64_16x16x4f64: lane l, register r hold row 4 r + l / 16,
// column l % 16.  So register b of a tile is exactly rows 4 b .. 4 b + 3 in the operand layout of the same
// instruction (k = l / 16), both as B and, transposed, as A: the four pivot rows of an elimination step go
// from registers to operands with no rearrangement, and one MFMA per tile does a step's rank-4 update.
//
// Elimination by blocks of four pivots.  Step t, pivot rows 4 t .. 4 t + 3 in tile row kb, with pivot block
// P = R^T R (4 x 4):
//   1. wave 0 brings tile (kb, kb) up to date first, takes P from its lanes and publishes R^-T (16 doubles),
//      while the other waves finish their updates of the step before; the owners publish the four raw rows;
//   2. after a barrier the waves scale the rows, U = R^-T [rows], 64 doubles per tile;
//   3. after a second barrier every tile (i, j), i >= kb, takes -= U_i^T U_j (in tile row kb only the rows
//      below the pivots).
// The registers keep the raw rows, which with the steps' R^-T is all that the back substitution needs
// (x_t = R^-1 R^-T (right-hand side - rows . x)); it goes by blocks of 16 rows.
//
// What bounds it is the chain of the steps: the 4 x 4 factor (four dependent reciprocal square roots), two LDS
// round trips and the MFMA latency, over a quarter of the columns.  So the pivot block is taken ahead by a wave
// with little else to do, and about nine tiles a wave leave room for four waves per SIMD.
#pragma once
#include "fbsde_device.hpp"

namespace fbsde {

typedef double spd_v4 __attribute__((ext_vector_type(4)));

// Tiles per side for n unknowns: the pivots are padded to a multiple of four, and the right-hand side's
// column comes right after them.
constexpr int spd_pivots(int n) { return (n + 3) / 4 * 4; }
constexpr int spd_tiles(int n) { return spd_pivots(n) / 16 + 1; }

// 1 / sqrt(x) from the hardware estimate by a cubic and a quadratic Newton step (relative error of the
// estimate below 2^-13, so the last step ends at rounding).
__device__ __forceinline__ double spd_rsqrt(double x) {
    double y = __builtin_amdgcn_rsq(x);
    double e = fma(-x * y, y, 1.0);
    y = fma(y * e, fma(0.375, e, 0.5), y);
    e = fma(-x * y, y, 1.0);
    return fma(0.5 * y, e, y);
}

__device__ __forceinline__ double spd_readlane(double x, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                            __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// Sum over the 16 lanes that share l / 16 (DPP row rotations); every lane gets it.
template <int ROR>
__device__ __forceinline__ double spd_ror(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x120 + ROR, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x120 + ROR, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double spd_row_sum(double x) {
    x += spd_ror<8>(x);
    x += spd_ror<4>(x);
    x += spd_ror<2>(x);
    x += spd_ror<1>(x);
    return x;
}

// Waves for T tiles per side (one for the diagonal, the others share the rest) and the waves per SIMD asked of
// the register allocator: the pairs that put the most blocks on a compute unit without spilling in the steps.
constexpr int spd_waves(int T) { return T <= 1 ? T : T <= 4 ? 2 : T <= 13 ? 4 : 8; }
constexpr int spd_occupancy(int T) { return T <= 4 ? 4 : T <= 8 ? 4 : T <= 10 ? 3 : 2; }

// LDS of one system.
template <int T>
struct SpdShared {
    double U[T * 64], Us[T * 64];   // a step's raw and scaled pivot rows
    double Ua[T * 64];              // the scaled rows negated, zero where the update must not reach (rows done)
    double Rt[4 * T * 16];          // R^-T of every step, row-major 4 x 4, lower triangle
    double x[T * 16];               // the right-hand side, then the solution
    double part[spd_waves(T) * 16];
    double D[T * 256];              // the diagonal tiles as the elimination leaves them
};

template <int T>
struct SpdSystem {
    static constexpr int NW = spd_waves(T);                   // a power of two
    static constexpr int NO = NW > 1 ? NW - 1 : 1;            // waves that share the tiles off the diagonal
    static constexpr int NOFF = T * (T - 1) / 2;              // tiles (i, j), i < j, row by row
    static constexpr int SLOTS = (NOFF + NO - 1) / NO;        // of them per wave: numbers s NO + wave - 1
    static constexpr int NTC = SLOTS / 2 + 1;
    static constexpr int GRP = 4;                             // slots whose operand loads are in flight at once
    uint32_t tc[NTC];   // wave-uniform tile coordinates of the slots, two a word: i | j << 8
    int nlive;          // slots that hold a tile (the others read in bounds and are never used)
    int wave, lane, g, c;   // g = lane / 16, c = lane % 16

    __device__ __forceinline__ int ti(int s) const { return (int)((tc[s >> 1] >> (16 * (s & 1))) & 255u); }
    __device__ __forceinline__ int tj(int s) const { return (int)((tc[s >> 1] >> (16 * (s & 1) + 8)) & 255u); }
    // Keeps the compiler from holding what it derives from the coordinates in scalar registers across the
    // steps (a few values per slot: it spilled hundreds).
    __device__ __forceinline__ void forget() {
#pragma unroll
        for (int q = 0; q < NTC; ++q) asm volatile("" : "+s"(tc[q]));
    }

    // id: a number of the block.  A block's wavefronts go to the SIMDs in order, and wave 0 has the pivot blocks
    // to do besides its tiles: where few blocks fit a compute unit (T >= 10) the roles are dealt by a hash of
    // the id, or the same SIMD would carry all of them (measured, 200 unknowns, 12800 systems: 2.93 ms against
    // 3.36; at 100 unknowns, four blocks a unit, 0.40 against 0.39 the other way).
    __device__ __forceinline__ void init(uint32_t id) {
        const int rot = (T >= 10) ? (int)((id * 2654435761u) >> 16 & (NW - 1)) : 0;
        wave = __builtin_amdgcn_readfirstlane(((threadIdx.x >> 6) + rot) & (NW - 1));
        lane = threadIdx.x & 63;
        g = lane >> 4;
        c = lane & 15;
        nlive = (wave == 0) ? 0 : (NOFF - (wave - 1) + NO - 1) / NO;
        int i = 0, j = wave;   // tile number wave - 1 of row 0 is (0, wave)
#pragma unroll
        for (int s = 0; s < 2 * NTC; ++s) {
            while (i < T && j >= T) { ++i; j += i + 1 - T; }
            const uint32_t code = (i < T - 1) ? (uint32_t)(i | (j << 8)) : 0u;
            tc[s >> 1] = (s & 1) ? (tc[s >> 1] | (code << 16)) : code;
            j += NO;
        }
#pragma unroll
        for (int q = 0; q < NTC; ++q) tc[q] = (uint32_t)__builtin_amdgcn_readfirstlane((int)tc[q]);
    }

    // R^-T of the 4 x 4 pivot block whose rows are `u` (register B of the diagonal tile); false where a pivot
    // is not positive.
    template <int B>
    static __device__ __forceinline__ bool pivot_block(double u, int lane, double* Rt) {
        const double p00 = spd_readlane(u, 4 * B), p01 = spd_readlane(u, 4 * B + 1),
                     p02 = spd_readlane(u, 4 * B + 2), p03 = spd_readlane(u, 4 * B + 3);
        const double p11 = spd_readlane(u, 16 + 4 * B + 1), p12 = spd_readlane(u, 16 + 4 * B + 2),
                     p13 = spd_readlane(u, 16 + 4 * B + 3);
        const double p22 = spd_readlane(u, 32 + 4 * B + 2), p23 = spd_readlane(u, 32 + 4 * B + 3);
        const double p33 = spd_readlane(u, 48 + 4 * B + 3);
        // one pivot after the other: a product of pivots (a 2 x 2 determinant for two at a time) leaves the range of
        // FP64 for matrices beyond 1e+-154, which sigma beyond 1e+-77 gives
        const double i0 = spd_rsqrt(p00);
        const double r01 = p01 * i0, r02 = p02 * i0, r03 = p03 * i0;
        const double q11 = fma(-r01, r01, p11), i1 = spd_rsqrt(q11);
        const double r12 = fma(-r01, r02, p12) * i1, r13 = fma(-r01, r03, p13) * i1;
        const double q22 = fma(-r12, r12, fma(-r02, r02, p22)), i2 = spd_rsqrt(q22);
        const double r23 = fma(-r12, r13, fma(-r02, r03, p23)) * i2;
        const double q33 = fma(-r23, r23, fma(-r13, r13, fma(-r03, r03, p33))), i3 = spd_rsqrt(q33);
        const double m10 = -r01 * i0 * i1;
        const double m20 = -fma(r02, i0, r12 * m10) * i2, m21 = -r12 * i1 * i2;
        const double m30 = -fma(r03, i0, fma(r13, m10, r23 * m20)) * i3, m31 = -fma(r13, i1, r23 * m21) * i3,
                     m32 = -r23 * i2 * i3;
        if (lane == 0) {   // the zeros above the diagonal are written once, by solve()
            Rt[0] = i0;
            Rt[4] = m10;  Rt[5] = i1;
            Rt[8] = m20;  Rt[9] = m21;  Rt[10] = i2;
            Rt[12] = m30; Rt[13] = m31; Rt[14] = m32;  Rt[15] = i3;
        }
        return p00 > 0.0 && q11 > 0.0 && q22 > 0.0 && q33 > 0.0;
    }

    // Step 2: every wave scales its share of the published rows, between two barriers.
    template <int B>
    __device__ __forceinline__ void scale(int kb, SpdShared<T>& sh) {
        __syncthreads();
        const double* R = sh.Rt + (4 * kb + B) * 16 + 4 * g;
        const double r0 = R[0], r1 = R[1], r2 = R[2], r3 = R[3];
        for (int j = kb + wave; j < T; j += NW) {
            const double* u = sh.U + 64 * j + c;
            const double us = fma(r3, u[48], fma(r2, u[32], fma(r1, u[16], r0 * u[0])));
            sh.Us[64 * j + lane] = us;
            sh.Ua[64 * j + lane] = (j == kb && (B == 3 || c < 4 * (B + 1))) ? 0.0 : -us;
        }
        __syncthreads();
    }

    template <int B>
    static __device__ __forceinline__ void back_step(int kb, int np, const spd_v4& d, double (&y)[4], int lane, int c,
                                                     SpdShared<T>& sh) {
        if (16 * kb + 4 * B >= np) return;
        const double* Rt = sh.Rt + (4 * kb + B) * 16;
        const double y0 = spd_readlane(y[B], 0), y1 = spd_readlane(y[B], 16), y2 = spd_readlane(y[B], 32),
                     y3 = spd_readlane(y[B], 48);
        const double z0 = Rt[0] * y0, z1 = fma(Rt[5], y1, Rt[4] * y0),
                     z2 = fma(Rt[10], y2, fma(Rt[9], y1, Rt[8] * y0)),
                     z3 = fma(Rt[15], y3, fma(Rt[14], y2, fma(Rt[13], y1, Rt[12] * y0)));
        const double x0 = fma(Rt[0], z0, fma(Rt[4], z1, fma(Rt[8], z2, Rt[12] * z3)));
        const double x1 = fma(Rt[5], z1, fma(Rt[9], z2, Rt[13] * z3));
        const double x2 = fma(Rt[10], z2, Rt[14] * z3);
        const double x3 = Rt[15] * z3;
        const int e = c - 4 * B;
        const double xc = (e == 0) ? x0 : (e == 1) ? x1 : (e == 2) ? x2 : (e == 3) ? x3 : 0.0;
#pragma unroll
        for (int r = 0; r < B; ++r) y[r] -= spd_row_sum(d[r] * xc);
        if (lane >= 4 * B && lane < 4 * B + 4) sh.x[16 * kb + lane] = xc;
    }

    // This lane's share of x^T A x for the symmetric matrix whose entries are load(row, column) and x in sh.x.
    template <typename Load>
    __device__ __forceinline__ double quadratic(Load&& load, const SpdShared<T>& sh) const {
        double a = 0.0, d = 0.0;
        auto tile = [&](int i, int j) {
            double t[4], q = 0.0;
#pragma unroll
            for (int r = 0; r < 4; ++r) t[r] = load(16 * i + 4 * r + g, 16 * j + c);
#pragma unroll
            for (int r = 0; r < 4; ++r) q = fma(sh.x[16 * i + 4 * r + g], t[r], q);
            return q * sh.x[16 * j + c];
        };
        if (wave == 0) {
#pragma unroll 2
            for (int q = 0; q < T; ++q) d += tile(q, q);
        } else {
            int i = 0, j = wave;   // the slots' coordinates again
#pragma unroll 2
            for (int s = 0; s < nlive; ++s) {
                while (j >= T) { ++i; j += i + 1 - T; }
                a += tile(i, j);
                j += NO;
            }
        }
        return d + 2.0 * a;
    }

    // ---- wave 0: the diagonal tiles, v[q] the one of tile row kb + q (moved down after each tile row, so that
    // every register index is a constant)
    template <int B>
    __device__ __forceinline__ bool publish_diag(const spd_v4& t, int kb, SpdShared<T>& sh) {
        sh.U[64 * kb + lane] = t[B];
        return pivot_block<B>(t[B], lane, sh.Rt + (4 * kb + B) * 16);
    }
    __device__ __forceinline__ void next_row(spd_v4 (&v)[T], int kb, SpdShared<T>& sh) {   // keeps the finished tile
#pragma unroll
        for (int r = 0; r < 4; ++r) sh.D[256 * kb + 64 * r + lane] = v[0][r];
#pragma unroll
        for (int q = 1; q < T; ++q) v[q - 1] = v[q];
    }
    template <int B>
    __device__ __forceinline__ bool step_diag(spd_v4 (&v)[T], int kb, bool more, SpdShared<T>& sh) {
        bool good = true;
        scale<B>(kb, sh);
        if (B == 3) next_row(v, kb, sh);
        const int kn = (B < 3) ? kb : kb + 1;   // tile row of the next step
        if (more) {
            v[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(sh.Ua[64 * kn + lane], sh.Us[64 * kn + lane], v[0], 0, 0, 0);
            good = publish_diag<(B + 1) & 3>(v[0], kn, sh);
        }
#pragma unroll
        for (int q0 = 1; q0 < T; q0 += GRP) {
            if (kn + q0 >= T) break;
            // tiles past the last one read in bounds and are never used
            double w[GRP];
#pragma unroll
            for (int q = q0; q < q0 + GRP; ++q)
                if (q < T) w[q - q0] = sh.Us[64 * min(kn + q, T - 1) + lane];
#pragma unroll
            for (int q = q0; q < q0 + GRP; ++q)
                if (q < T) v[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(-w[q - q0], w[q - q0], v[q], 0, 0, 0);
        }
        return good;
    }
    template <typename Load, typename Map, typename Diag, typename Rhs>
    __device__ __forceinline__ bool solve_diag(Load&& load, Map&& map, Diag&& diag, Rhs&& rhs, int np, int col, SpdShared<T>& sh) {
        spd_v4 v[T];
#pragma unroll
        for (int q = 0; q < T; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) v[q][r] = load(16 * q + 4 * r + g, 16 * q + c);
#pragma unroll
        for (int q = 0; q < T; ++q) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 16 * q + 4 * r + g, j = 16 * q + c;
                v[q][r] = map(v[q][r], i, j) + ((i == j) ? diag(i) : 0.0);
                if (q == (col >> 4) && j == col) v[q][r] = rhs(i);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        bool good = publish_diag<0>(v[0], 0, sh);
        for (int kb = 0; 16 * kb < np; ++kb) {
            const int left = np - 16 * kb;
            good &= step_diag<0>(v, kb, left > 4, sh);
            if (left > 4) good &= step_diag<1>(v, kb, left > 8, sh);
            if (left > 8) good &= step_diag<2>(v, kb, left > 12, sh);
            if (left > 12) good &= step_diag<3>(v, kb, left > 16, sh);
            else next_row(v, kb, sh);
        }
        // back substitution, this wave's part: the 16 rows of a tile row, once the others have summed theirs
        const int kc = col >> 4;
        if (c == (col & 15) && 16 * kc < np) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (16 * kc + 4 * r + g < np) sh.x[16 * kc + 4 * r + g] = sh.D[256 * kc + 64 * r + lane];
        }
        __syncthreads();
        for (int kb = (np - 1) / 16; kb >= 0; --kb) {
            __syncthreads();
            spd_v4 d;
            double y[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                d[r] = sh.D[256 * kb + 64 * r + lane];
                y[r] = sh.x[16 * kb + 4 * r + g];
#pragma unroll
                for (int w = 1; w < NW; ++w) y[r] -= sh.part[16 * w + 4 * r + g];
            }
            back_step<3>(kb, np, d, y, lane, c, sh);
            back_step<2>(kb, np, d, y, lane, c, sh);
            back_step<1>(kb, np, d, y, lane, c, sh);
            back_step<0>(kb, np, d, y, lane, c, sh);
            __syncthreads();
        }
        return good;
    }

    // ---- the other waves: their share of the tiles off the diagonal
    // mrow: the wave's slots in the tile row of the published step
    template <int B>
    __device__ __forceinline__ void publish_off(const spd_v4 (&v)[SLOTS], uint32_t mrow, SpdShared<T>& sh) {
#pragma unroll
        for (int s0 = 0; s0 < SLOTS; s0 += GRP)
            if (mrow >> s0 & ((1u << GRP) - 1u)) {
#pragma unroll
                for (int s = s0; s < s0 + GRP && s < SLOTS; ++s)
                    if (mrow >> s & 1u) sh.U[64 * tj(s) + lane] = v[s][B];
            }
    }
    __device__ __forceinline__ uint32_t row_mask(int kb) const {
        uint32_t m = 0u;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) m |= (s < nlive && ti(s) == kb) ? 1u << s : 0u;
        return m;
    }
    template <int B>
    __device__ __forceinline__ void step_off(spd_v4 (&v)[SLOTS], int kb, bool more, uint32_t& mrow, SpdShared<T>& sh) {
        scale<B>(kb, sh);
        forget();
#pragma unroll
        for (int s0 = 0; s0 < SLOTS; s0 += GRP) {
            const int last = s0 + GRP - 1 < SLOTS ? s0 + GRP - 1 : SLOTS - 1;
            // tile rows are in order: below the pivots' row the whole group is finished
            if (last < nlive && ti(last) < kb + (B == 3)) continue;
            // no branch within a group, so that its loads are all in flight before the first MFMA
            double a[GRP], b[GRP];
#pragma unroll
            for (int s = s0; s <= last; ++s) {
                a[s - s0] = sh.Ua[64 * ti(s) + lane];
                b[s - s0] = sh.Us[64 * tj(s) + lane];
            }
#pragma unroll
            for (int s = s0; s <= last; ++s)
                v[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s - s0], b[s - s0], v[s], 0, 0, 0);
        }
        if (B == 3) mrow = row_mask(kb + 1);
        if (more) publish_off<(B + 1) & 3>(v, mrow, sh);
    }
    template <typename Load, typename Map, typename Rhs>
    __device__ __forceinline__ void solve_off(Load&& load, Map&& map, Rhs&& rhs, int np, int col, SpdShared<T>& sh) {
        spd_v4 v[SLOTS];
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
#pragma unroll
            for (int r = 0; r < 4; ++r) v[s][r] = load(16 * ti(s) + 4 * r + g, 16 * tj(s) + c);
        forget();
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[s][r] = map(v[s][r], 16 * ti(s) + 4 * r + g, 16 * tj(s) + c);
            if (tj(s) == (col >> 4) && c == (col & 15)) {
#pragma unroll
                for (int r = 0; r < 4; ++r) v[s][r] = rhs(16 * ti(s) + 4 * r + g);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        forget();
        uint32_t mrow = row_mask(0);
        publish_off<0>(v, mrow, sh);
        for (int kb = 0; 16 * kb < np; ++kb) {
            const int left = np - 16 * kb;
            step_off<0>(v, kb, left > 4, mrow, sh);
            if (left > 4) step_off<1>(v, kb, left > 8, mrow, sh);
            if (left > 8) step_off<2>(v, kb, left > 12, mrow, sh);
            if (left > 12) step_off<3>(v, kb, left > 16, mrow, sh);
        }
        // back substitution, these waves' part: the right-hand side, then the sums over the solved columns
        if (c == (col & 15)) {
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
                if (s < nlive && tj(s) == (col >> 4)) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int i = 16 * ti(s) + 4 * r + g;
                        if (i < np) sh.x[i] = v[s][r];
                    }
                }
        }
        __syncthreads();
        for (int kb = (np - 1) / 16; kb >= 0; --kb) {
            forget();
            double q[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
                if (s < nlive && ti(s) == kb) {
                    const double xc = sh.x[16 * tj(s) + c];
#pragma unroll
                    for (int r = 0; r < 4; ++r) q[r] = fma(v[s][r], xc, q[r]);
                }
#pragma unroll
            for (int r = 0; r < 4; ++r) q[r] = spd_row_sum(q[r]);
            const double qs = (c == 0) ? q[0] : (c == 1) ? q[1] : (c == 2) ? q[2] : q[3];
            if (c < 4) sh.part[16 * wave + 4 * c + g] = qs;
            __syncthreads();
            __syncthreads();
        }
    }

    // Solves the system of np (a multiple of four) unknowns whose entry (i, j) is map(load(i, j), i, j), plus
    // diag(i) on the diagonal, for the right-hand side rhs(i), held in column `col` >= np; i and j run up to
    // 16 T.  `load` only reads memory, so that a tile's loads are all in flight together.  The solution is in
    // sh.x, zero beyond np, for all threads.  Returns false, on wave 0, where a pivot was not positive.  The
    // functions do not read sh.
    template <typename Load, typename Map, typename Diag, typename Rhs>
    __device__ __forceinline__ bool solve(Load&& load, Map&& map, Diag&& diag, Rhs&& rhs, int np, int col,
                                          SpdShared<T>& sh) {
        bool good = true;
        // zeros above the diagonals of R^-T; the steps' barriers put them before their first use
        for (int i = threadIdx.x; i < 4 * T * 16; i += 64 * NW)
            if ((i >> 2 & 3) < (i & 3)) sh.Rt[i] = 0.0;
        for (int i = np + threadIdx.x; i < 16 * T; i += 64 * NW) sh.x[i] = 0.0;   // the sums run over whole tiles
        if (wave == 0) good = solve_diag(load, map, diag, rhs, np, col, sh);
        else if constexpr (NW > 1) solve_off(load, map, rhs, np, col, sh);
        return good;
    }
};

}  // namespace fbsde
