// Host-side helpers shared by the translation units of libfbsde (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <type_traits>

#include "fbsde.h"
#include "fbsde_device.hpp"

namespace fbsde {
namespace host {


constexpr int NS = 10;   // per-point FP64 scalars (see k_moments_finish and k_level_finish)

struct Plan {
    int64_t d, M, N;
    int ld, Q, TEAM, BS, TPW, nchunk, rows_per_chunk;
    size_t esz;
    int maxit;   // CG iterations per point and level at most (sizes the device loop's work queues)
    int direct;  // the forward levels' solve: DIRECT_NONE (CG), DIRECT_DUAL (M x M), DIRECT_PRIMAL (d x d)
    int dsplit;  // slices of the direct solve's Gram matrix
    int least_chunks;   // chunks per point that a smaller workspace may bring the plan down to
};

enum { DIRECT_NONE = 0, DIRECT_DUAL = 1, DIRECT_PRIMAL = 2 };
constexpr int DIRECT_MAXD = 128;   // largest d of the primal direct solve
// Smallest ridge of the primal direct solve.  A narrow kernel's weights leave the design with fewer particles than
// coordinates, and what keeps the d x d matrix positive is the ridge alone: a pivot is positive for certain while the
// ridge over the largest diagonal entry is above d (d + 1) 2^-53 (1.8e-12 at d = 128), and that entry reaches some 20
// times the ridge's own scale s^2 t, d times it under x-dependent coefficients.  Below, the CG, which needs no
// positive pivot (seen at kernel factors of 0.03 to 0.1: no point fails at 1e-12 and above, up to 15 of 300 at 1e-15,
// half of them at 1e-18; from 1e-8 up the direct solve's error is at or below the CG's at every one tried).
constexpr double DIRECT_MIN_RIDGE = 1e-8;

inline int64_t round_up(int64_t a, int64_t b) { return (a + b - 1) / b * b; }

inline int check_problem(const fbsde_problem* pb, int64_t P) {
    if (!pb || P < 0) return FBSDE_EINVAL;
    if (pb->d < 1 || pb->M < 2 || pb->N < 1) return FBSDE_EINVAL;
    if (!(pb->T > 0.0) || !(pb->s > 0.0)) return FBSDE_EINVAL;
    if (pb->f_kind < FBSDE_F_ZERO || pb->f_kind > FBSDE_F_LOG_POT) return FBSDE_EINVAL;
    if (pb->g_kind < FBSDE_G_QUAD || pb->g_kind > FBSDE_G_CASE2) return FBSDE_EINVAL;
    if ((pb->g_kind == FBSDE_G_AFFINE || pb->g_kind == FBSDE_G_LOGISTIC) && !pb->gvec) return FBSDE_EINVAL;
    if (!(pb->eps_h >= 0.0) || !(pb->ridge_rel >= 0.0)) return FBSDE_EINVAL;
    if (pb->ridge_rel == 0.0 && pb->M <= pb->d + 1) return FBSDE_EINVAL;
    if (pb->newton_iters < 1 || pb->cg_maxit < 1 || !(pb->cg_rtol >= 0.0)) return FBSDE_EINVAL;
    if (pb->prec != FBSDE_F64 && pb->prec != FBSDE_F32C) return FBSDE_EINVAL;
    if (pb->shared_dw != 0 && pb->shared_dw != 1) return FBSDE_EINVAL;
    if (pb->solver != FBSDE_SOLVER_AUTO && pb->solver != FBSDE_SOLVER_CG) return FBSDE_EINVAL;
    // grid.y carries the point index
    if (pb->M > (int64_t)1 << 30 || pb->N > (int64_t)1 << 30 || P > 65535) return FBSDE_EINVAL;
    return FBSDE_OK;
}

// CG stopping tolerance actually used.  In FP32C with a rank-deficient centred design (M <= d + 1) the
// right-hand side carries FP32 rounding in the ridge-only null space; a test tighter than that rounding
// makes CG resolve it, scaled by 1/lam, into the slope: the tolerance is held at 1e-7 or above there.
inline double cg_rtol_of(const fbsde_problem* pb) {
    if (pb->prec == FBSDE_F32C && pb->M <= pb->d + 1) return std::max(pb->cg_rtol, 1e-7);
    return pb->cg_rtol;
}

// Launch timer records (fbsde_launch_timer): begin returns a record index or -1 when the timer is off.
long timer_begin(hipStream_t st, double work, int kind);
void timer_end(long i, hipStream_t st);

// Launch shapes recorded by fbsde_autotune (process-wide table keyed by precision, d, M and P).
bool tuned_shape(const fbsde_problem* pb, int64_t P, int& team, int& nchunk);

// Groups of four coordinates per lane for q needed: 1, 2, 4, 8, and 5 on the FP32 state (rows of
// 4097-5120 coordinates on four-wave teams, 8193-10240 on eight: no idle lane groups, and fewer registers
// than 8 groups).
inline int groups_per_lane(int q, int esz) {
    return (q <= 1) ? 1 : (q <= 2) ? 2 : (q <= 4) ? 4 : (q <= 5 && esz == 4) ? 5 : 8;
}

// Re-shape a plan: team width `team` (groups per lane recomputed) and `nchunk` chunks per point.
// Returns false if the team cannot hold the row within the per-lane register budget.
inline bool shape_plan(Plan& pl, int team, int nchunk) {
    const int groups = pl.ld / 4;
    const int qmax = (pl.esz == 8) ? 4 : 8;
    if (team < 1 || team > 16 || (team & (team - 1)) || nchunk < 1) return false;
    const int q = (groups + 64 * team - 1) / (64 * team);
    if (q > qmax) return false;
    pl.TEAM = team;
    pl.Q = groups_per_lane(q, pl.esz);
    pl.BS = 64 * std::max(pl.TEAM, 4);
    pl.TPW = pl.BS / (64 * pl.TEAM);
    pl.rows_per_chunk = (int)((pl.M + nchunk - 1) / nchunk);
    pl.nchunk = (int)((pl.M + pl.rows_per_chunk - 1) / pl.rows_per_chunk);
    return true;
}

// Blocks of the CG loop that a compute unit holds at once, by its registers as compiled (k_cg_loop over the state's
// and the arithmetic's type, groups per lane and team width).
inline int cg_blocks_per_cu(const Plan& pl, bool r64) {
    if (pl.BS > 256) return 1;
    if (pl.Q == 1) return 5;
    if (pl.esz == 8) return (pl.Q == 2) ? 4 : 2;
    if (pl.Q == 2) return r64 ? 4 : 5;
    if (pl.Q == 4) return r64 ? 3 : 4;
    if (pl.Q == 5) return (pl.TEAM == 1 && !r64) ? 3 : 2;
    return (pl.TEAM == 2) ? 1 : 2;
}

inline int make_plan(const fbsde_problem* pb, int64_t P, Plan& pl) {
    pl.d = pb->d; pl.M = pb->M; pl.N = pb->N;
    pl.maxit = std::max(1, (int)pb->cg_maxit);
    // The direct dual solve where the cloud is small (the Gram kernel holds the tiles of at most 128 rows in registers)
    // and not much thinner than d.  The line at M = d / 8 was drawn for a solve of one block a point, which was slower
    // than the CG beyond it; the present one is the faster at every size tried (a level, 64 points, M = 100: FP64 d =
    // 500 141 against 656 us, d = 1000 186 against 727, d = 4000 455 against 1605; FP32C 133 and 368, 163 and 383, 444
    // and 736), so nothing would be lost by moving it.
    pl.direct = DIRECT_NONE;
    if (pb->solver == FBSDE_SOLVER_AUTO && !pb->shared_dw && pb->ridge_rel > 0.0 && pb->cg_fixed_iters == 0) {
        if (pb->M <= FBSDE_DUAL_MAXM && pb->M <= pb->d + 1 && 8 * pb->M >= pb->d) pl.direct = DIRECT_DUAL;
        // the direct primal solve where d is small: one read of the cloud instead of one per iteration
        // (FP64, a whole solve: one point at d = 100, M = 512, N = 5 2.67 -> 0.39 ms; 512 points at d = 100,
        // M = 1024, N = 20 80.1 -> 12.7 ms).  A cap below d asks for fewer iterations than an exact solve may take: it
        // keeps the CG.
        else if (pb->M > pb->d + 1 && pb->d <= DIRECT_MAXD && pb->cg_maxit >= pb->d && pb->ridge_rel >= DIRECT_MIN_RIDGE)
            pl.direct = DIRECT_PRIMAL;
    }
    pl.esz = (pb->prec == FBSDE_F64) ? 8 : 4;
    pl.ld = (int)round_up(pb->d, (pl.esz == 8) ? 16 : 32);
    const int groups = pl.ld / 4;
    const int qmax = (pl.esz == 8) ? 4 : 8;
    pl.TEAM = 0;
    for (int team = 1; team <= 16; team *= 2) {
        const int q = (groups + 64 * team - 1) / (64 * team);
        if (q <= qmax) {
            pl.TEAM = team;
            pl.Q = groups_per_lane(q, pl.esz);
            break;
        }
    }
    if (pl.TEAM == 0) return FBSDE_EINVAL;   // d beyond 16384 (FP64) / 32768 (FP32C)
    pl.BS = 64 * std::max(pl.TEAM, 4);
    pl.TPW = pl.BS / (64 * pl.TEAM);
    // Chunks per point, 16 rows each at least (8 on teams of eight waves and more).
    // Up to CG_MAXQ points, a queue each: one work item per block that the chip holds at once.  A point's next
    // iteration starts when all its items are done, so a part-empty second round costs as much as a full one, and
    // smaller items cost a partial vector and an arrival each.  Two levels, two items a block but at most 128 chunks
    // -> now, stealing as it is: d = 5544, M = 2965, 7 points 17.2 -> 15.8 ms; d = 2279, M = 3589, 5 points, FP64 30.6 ->
    // 24.6; d = 10^4, M = 1024, 16 points 8.4 -> 7.4; d = 1000, M = 4096, 16 points 3.9 -> 2.95; d = 2718, M = 2778, 25
    // points 201 -> 183 (before either change 186); d = 300, M = 65536, 3 points 3.08 -> 2.46.  At most 512 (one point,
    // d = 300, M = 65536, FP64 2.66 ms, with 1024 2.80).
    // More points share their queues and leave them one by one: two items a block, at most 128 chunks (64 points, d =
    // 1000, M = 4096: FP32C 9.7 against 9.3 ms with one, FP64 31.4 against 30.6; 150 points, d = 400, M = 900 13.1
    // against 13.4).
    // At least four chunks, but no more than 4096 items in all and, beyond ld = 1024, of 64 rows: beyond 1024 points
    // four cost 1.05 to 1.3 times the time (three levels: d = 200, M = 300, 8192 points 121 ms with one chunk, 137 with
    // four; d = 1000, M = 64, 16384 points 57 and 72) and the partial sums of four (d = 1000, M = 64, 65535 points 38.5 GB
    // and 44.0); 624 points at d = 3559, M = 182 13.3 ms with two and 13.9 with four.
    const bool r64 = pl.esz == 4 && pb->M <= pb->d + 1;   // FP64 arithmetic on the FP32 state (run_level)
    const int64_t np = std::max<int64_t>(P, 1), min_rows = (pl.TEAM >= 8) ? 8 : 16;
    const int64_t held = 256 * (int64_t)cg_blocks_per_cu(pl, r64);
    // Levels solved directly have no CG items, only the moments' and the reversal's rows: as for more points (8 points,
    // M = 10^5, d = 128: 128 chunks 348 and 168 us, 160 chunks 390 and 185).
    const int64_t per_point = (np <= CG_MAXQ && !pl.direct) ? std::min<int64_t>(held / np, 512)
                                                            : std::max<int64_t>(std::min<int64_t>(2 * held / np, 128), 512 / np);
    // 4096 items in all, 64 rows a chunk beyond ld = 1024: no more than this is asked of a workspace that is smaller
    // than the plan's own
    const int64_t few = std::min<int64_t>({(4096 + np - 1) / np, pb->M / (2 * pl.TPW), pb->M / ((pl.ld <= 1024) ? 16 : 64)});
    int64_t nchunk = std::max<int64_t>(per_point, std::min<int64_t>(4, few));
    nchunk = std::max<int64_t>(1, std::min<int64_t>(nchunk, std::min<int64_t>(pb->M / (2 * pl.TPW), pb->M / min_rows)));
    const auto chunks = [&](int64_t n) {
        pl.rows_per_chunk = (int)((pb->M + n - 1) / n);
        pl.nchunk = (int)((pb->M + pl.rows_per_chunk - 1) / pl.rows_per_chunk);
    };
    chunks(std::max<int64_t>(1, std::min<int64_t>(nchunk, few)));
    pl.least_chunks = pl.nchunk;
    chunks(nchunk);
    // a shape chosen by the autotuner: never more chunks than the default, so workspaces sized
    // before the tuning still fit
    int tt, tn;
    if (P > 0 && tuned_shape(pb, P, tt, tn)) {
        Plan t = pl;
        if (tn <= pl.nchunk && shape_plan(t, tt, tn)) pl = t;
    }
    // slices of the direct solve's contraction: about two blocks a compute unit in all (as many as are resident),
    // at least 32 indices each, at most 32 (each costs a partial of the whole triangle); with more points than
    // units, up to four slices where that leaves the units idle for less of the last round
    const int64_t len = (pl.direct == DIRECT_PRIMAL) ? pl.M : pl.ld;
    int64_t split = std::max<int64_t>(1, 512 / np);
    if (np > 256)
        for (int64_t n = 2; n <= 4; ++n)
            if (10 * ((np * n + 255) / 256) * split < 9 * ((np * split + 255) / 256) * n) split = n;
    pl.dsplit = (int)std::max<int64_t>(1, std::min<int64_t>({split, (len + 31) / 32, 32}));
    return FBSDE_OK;
}

template <typename S, typename Fn>
void dispatch(int Q, int TEAM, Fn&& fn) {
#define FB_CASE(QQ, TT) \
    case QQ * 100 + TT: fn(std::integral_constant<int, QQ>{}, std::integral_constant<int, TT>{}); return;
    switch (Q * 100 + TEAM) {
        FB_CASE(1, 1) FB_CASE(1, 2) FB_CASE(1, 4) FB_CASE(1, 8) FB_CASE(1, 16)
        FB_CASE(2, 1) FB_CASE(2, 2) FB_CASE(2, 4) FB_CASE(2, 8) FB_CASE(2, 16)
        FB_CASE(4, 1) FB_CASE(4, 2) FB_CASE(4, 4) FB_CASE(4, 8) FB_CASE(4, 16)
        default: break;
    }
    if constexpr (std::is_same<S, float>::value) {
        switch (Q * 100 + TEAM) {
            FB_CASE(5, 1) FB_CASE(5, 2) FB_CASE(5, 4) FB_CASE(5, 8) FB_CASE(5, 16)
            FB_CASE(8, 1) FB_CASE(8, 2) FB_CASE(8, 4) FB_CASE(8, 8) FB_CASE(8, 16)
            default: break;
        }
    }
#undef FB_CASE
}

struct Keys { uint32_t k0, k1; };
inline Keys keys_of(const fbsde_problem* pb) {
    return {(uint32_t)(pb->seed & 0xFFFFFFFFull), (uint32_t)((pb->seed >> 32) ^ (uint64_t)pb->instance)};
}
inline FSpec fspec_of(const fbsde_problem* pb) {
    if (pb->f_kind == FBSDE_F_HJ_SINK) return {pb->f_kind, pb->fp[0], 1.0 / (pb->s * pb->s)};
    return {pb->f_kind, pb->fp[0], pb->fp[1], pb->fp[2]};
}
// f depends on x (a source term): only the per-point forward paths evaluate it, at the particles'
// positions.
inline bool f_depends_on_x(const fbsde_problem* pb) {
    return pb->f_kind == FBSDE_F_HJ_SINK || pb->f_kind == FBSDE_F_LOG_POT;
}
// A family only the per-point forward paths evaluate: f depends on x, or g needs the product of the
// coordinates (the Case 2 terminal value, formed in the forward sweep of the per-point form).
inline bool per_point_forward_only(const fbsde_problem* pb) {
    return f_depends_on_x(pb) || pb->g_kind == FBSDE_G_CASE2;
}

inline int last_error() { return (hipGetLastError() == hipSuccess) ? FBSDE_OK : FBSDE_EHIP; }


// The direct level solve (fbsde_direct.hip): its buffers, and the launches that leave the slope, at the scale
// of k_moments_finish, in x.
size_t direct_part_bytes(const Plan& pl, int64_t P);
size_t direct_coef_bytes(const Plan& pl, int64_t P);
template <typename S>
int direct_solve(const Plan& pl, int64_t P, const S* W, int64_t ldw, double s, const double* Wbar, const double* w,
                 const double* Y, const double* r, const double* scal, double* part, double* coef, double* x, int* iscal,
                 uint32_t* status, hipStream_t st);

// Entry points of the other translation units.
size_t shared_workspace_bytes(const fbsde_problem* pb, int64_t P, int32_t flags);
int solve_shared(const fbsde_problem* pb, int64_t P, const double* x0, double* u, double* grad, uint32_t* status,
                 void* ws, size_t ws_bytes, int32_t flags, hipStream_t st);
int backward_shared(const fbsde_problem* pb, int64_t P, const double* x0, const double* u_bar, double* x0_bar,
                    double* gp_bar, double* fp_bar, uint32_t* status, void* ws, size_t ws_bytes, hipStream_t st);
// Newton adjoint of a level and the parameter sums (core translation unit owns these kernels).
void adj_newton(const fbsde_problem* pb, int64_t P, double* G, const double* w_prev, int64_t w_stride,
                const double* psc, int nchunk, const double* Yk, const double* tscal_k, const double* u_bar,
                double* cbar, double* adj, int init, int terminal, uint32_t* status, hipStream_t st);
void adj_params(const double* adj, int64_t P, double* gp_bar, double* fp_bar, hipStream_t st);
int tape_tag_of(const fbsde_problem* pb, int64_t P);
// W_{k+1} = W_k + sqrt(dt) xi_k on a single shared cloud (k = 0: from W_0 = 0).
template <typename S>
void shared_advance(const fbsde_problem* pb, const Plan& pl1, int k, S* W, hipStream_t st);
// Forward sweep / reversal of a single shared cloud (core translation unit owns these kernels).
template <typename S>
void shared_forward(const fbsde_problem* pb, const Plan& pl1, S* W, double* Yscratch, double* rn2, uint32_t* status,
                    hipStream_t st);
template <typename S>
void shared_reverse(const fbsde_problem* pb, const Plan& pl1, int k, S* W, const double* ax_dummy, const double* scal,
                    double* Yscratch, double* rn2, uint32_t* status, hipStream_t st);
void clear_status(uint32_t* status, int64_t P, hipStream_t st);
// Capture what body enqueues (on the stream it is given) into a graph, as fbsde_graph_capture does.
int capture_graph(const std::function<int(hipStream_t)>& body, hipStream_t stream, fbsde_graph* out);
// Divisor of the chip's block slots that a CG loop launch from this host thread asks for (1 by default).
extern thread_local int loop_share;
// fbsde_solve for one tile of a batched call; reset_counts = false adds its CG traffic to the count the
// arena already holds (the per-point form keeps it in the loop control at offset 0 of the workspace).
int solve_tile(const fbsde_problem* pb, int64_t P, const double* x0, double* u, double* grad, uint32_t* status,
               void* ws, size_t ws_bytes, int32_t flags, bool reset_counts, hipStream_t st);
// Device address of the algorithmic CG-product byte count in a per-point workspace.
unsigned long long* cg_bytes_counter(void* ws);
// fbsde_solve_backward without the read-back of the tape's tag, for a caller that has just enqueued the
// forward solve with the tape on the same stream and workspace (the batched schedule): no stream wait.
int solve_backward_after_forward(const fbsde_problem* pb, int64_t P, const double* x0, const double* u_bar,
                                 double* x0_bar, double* gp_bar, double* fp_bar, uint32_t* status, void* ws,
                                 size_t ws_bytes, hipStream_t st);
void set_int(int* a, int v, hipStream_t st);
// The per-point solve (fbsde_solve, no tape) with a step run after the forward sweep that may rewrite the
// terminal values Y [P][M] from the state W [P][M][ldw] (a constant diffusion matrix enters here);
// per_point_workspace_bytes is its workspace.
using TerminalStep = std::function<int(const void* W, int64_t ldw, double* Y, hipStream_t)>;
size_t per_point_workspace_bytes(const fbsde_problem* pb, int64_t P, int32_t flags);
// The least it runs in, with fewer work items and Gram slices (fit_plan).
size_t per_point_least_bytes(const fbsde_problem* pb, int64_t P, int32_t flags);
int solve_per_point_terminal(const fbsde_problem* pb, int64_t P, const double* x0, double* u, double* grad,
                             uint32_t* status, void* ws, size_t ws_bytes, int32_t flags, int32_t* cg_iters_out,
                             hipStream_t st, const TerminalStep& terminal);
// The reverse mode of that solve with the terminal stage changed the same way: `before` fills qpre [P][M]
// (the argument of g per particle) from the state W_N, the terminal adjoint then reads it, its x0 adjoint is
// formed without the W-column term, and `after` adds that term from the W-column sums (part, summed over
// its first vchunks chunk slots of ld) to x0_bar.
struct AdjTerminalHooks {
    std::function<int(const void* W, int64_t ldw, hipStream_t)> before;
    double* qpre;
    std::function<int(const double* part, int nchunk, int vchunks, int ld, double* x0_bar, hipStream_t)> after;
};
int solve_per_point_backward_terminal(const fbsde_problem* pb, int64_t P, const double* x0, const double* u_bar,
                                      double* x0_bar, double* gp_bar, double* fp_bar, uint32_t* status, void* ws,
                                      size_t ws_bytes, int32_t* cg_iters_out, hipStream_t st,
                                      const AdjTerminalHooks& hooks);

}  // namespace host
}  // namespace fbsde
