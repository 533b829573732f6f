// Launches of the direct level solves (fbsde_direct.hpp): a translation unit of its own, since the factorisation
// is instantiated per system size.
#include "fbsde_host.hpp"
#include "fbsde_direct.hpp"

namespace fbsde {
namespace host {

namespace {

int direct_n(const Plan& pl) { return (int)((pl.direct == DIRECT_PRIMAL) ? pl.d : pl.M); }

template <typename S, int NT, bool PRIMAL>
void gram(const Plan& pl, int64_t P, const S* W, int64_t ldw, double s, const double* Wbar, const double* w, double* part,
          int nsplit, hipStream_t st) {
    const int64_t len = PRIMAL ? pl.M : pl.ld;
    const int slice = (int)round_up((len + nsplit - 1) / nsplit, GRAM_SLICE);
    hipLaunchKernelGGL((k_gram<S, NT, PRIMAL ? GRAM_PRIMAL : GRAM_DUAL>), dim3(nsplit, (unsigned)P), dim3(256), 0, st, W,
                       ldw, (int)pl.M, pl.ld, direct_n(pl), slice, s, Wbar, w, part, nullptr);
}

}  // namespace

size_t direct_part_bytes(const Plan& pl, int64_t P) {
    return (size_t)P * pl.dsplit * gram_entries(direct_n(pl)) * 8;
}
size_t direct_coef_bytes(const Plan& pl, int64_t P) {
    return (pl.direct == DIRECT_DUAL) ? (size_t)P * (pl.M + 1) * 8 : 0;
}

template <typename S>
int direct_solve(const Plan& pl, int64_t P, const S* W, int64_t ldw, double s, const double* Wbar, const double* w,
                 const double* Y, const double* r, const double* scal, double* part, double* coef, double* x, int* iscal,
                 uint32_t* status, hipStream_t st) {
    const bool primal = pl.direct == DIRECT_PRIMAL;
    const int n = direct_n(pl), nt = (n + 15) / 16, nsplit = pl.dsplit;
    switch (nt) {
#define FB_GRAM(NT)                                                                            \
    case NT:                                                                                   \
        if (primal) gram<S, NT, true>(pl, P, W, ldw, s, Wbar, w, part, nsplit, st);             \
        else gram<S, NT, false>(pl, P, W, ldw, s, Wbar, w, part, nsplit, st);                   \
        break;
        FB_GRAM(1) FB_GRAM(2) FB_GRAM(3) FB_GRAM(4) FB_GRAM(5) FB_GRAM(6) FB_GRAM(7) FB_GRAM(8)
#undef FB_GRAM
        default: return FBSDE_EINVAL;
    }
    const int64_t ne = gram_entries(n);
    if (nsplit > 1)
        hipLaunchKernelGGL(k_direct_fold, dim3((unsigned)((ne + 255) / 256), (unsigned)P), dim3(256), 0, st, part, nsplit, ne);
    switch (spd_tiles(n)) {
#define FB_SOLVE(T)                                                                                                     \
    case T:                                                                                                             \
        if (primal)                                                                                                     \
            hipLaunchKernelGGL((k_direct_solve<T, true>), dim3((unsigned)P), dim3(64 * spd_waves(T)), 0, st, part,      \
                               nsplit * ne, n, pl.ld, s, w, Y, r, scal, NS, coef, x, iscal, status);                \
        else                                                                                                            \
            hipLaunchKernelGGL((k_direct_solve<T, false>), dim3((unsigned)P), dim3(64 * spd_waves(T)), 0, st, part,     \
                               nsplit * ne, n, pl.ld, s, w, Y, r, scal, NS, coef, x, iscal, status);                \
        break;
        FB_SOLVE(1) FB_SOLVE(2) FB_SOLVE(3) FB_SOLVE(4) FB_SOLVE(5) FB_SOLVE(6) FB_SOLVE(7) FB_SOLVE(8) FB_SOLVE(9)
#undef FB_SOLVE
        default: return FBSDE_EINVAL;
    }
    if (!primal)
        hipLaunchKernelGGL((k_direct_alpha<S>), dim3((unsigned)((pl.ld + 63) / 64), (unsigned)P), dim3(256), 0, st, coef,
                           (int)pl.M, W, ldw, pl.ld, Wbar, x);
    return last_error();
}

template int direct_solve<double>(const Plan&, int64_t, const double*, int64_t, double, const double*, const double*,
                                  const double*, const double*, const double*, double*, double*, double*, int*, uint32_t*,
                                  hipStream_t);
template int direct_solve<float>(const Plan&, int64_t, const float*, int64_t, double, const double*, const double*,
                                 const double*, const double*, const double*, double*, double*, double*, int*, uint32_t*,
                                 hipStream_t);

}  // namespace host
}  // namespace fbsde
