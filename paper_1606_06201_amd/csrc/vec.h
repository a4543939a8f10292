// Launchers of the dimension-independent kernels (vec.hip).
#pragma once
#include "common.h"

namespace ipmg {

void vdot(hipStream_t st, const double* a, const double* b, int64_t n, const Red& red, int sidx, const int* gate);
template <typename T>
void vdot_beta(hipStream_t st, const double* r, const T* y, int64_t n, const Red& red, const int* gate);
template <typename T>
void vdot_store(hipStream_t st, const double* r, const T* y, int64_t n, const Red& red, int sidx, const int* gate);
template <typename T>
void vpcg_update(hipStream_t st, double* z, double* r, const double* p, const double* q, T* rT, int64_t n,
                 const Red& red, const int* gate);   // z may be null; block partials of ||r||^2 ...
// ... summed, done flag; zpend: z was left out (flags[F_ZPEND] set for the next step)
void vpcg_update_fin(hipStream_t st, int64_t n, const Red& red, const int* gate, bool zpend = false);
unsigned vpcg_update_blocks(int64_t n);   // partials vpcg_update writes
void vpcg_update_fin_nb(hipStream_t st, unsigned nblocks, const Red& red, const int* gate, bool zpend);
// z += alpha p if flags[F_ZPEND], then the flag cleared (after the PCG step loop).
void vzflush(hipStream_t st, double* z, const double* p, int64_t n, const Red& red);
template <typename T>
void vpcg_dir(hipStream_t st, double* p, const T* y, int64_t n, const Red& red, int first, const int* gate);
void vsub_norm(hipStream_t st, const double* a, const double* b, double* out, int64_t n, const Red& red, int sidx);
void vmask_copy(hipStream_t st, const double* src, double* dst, int64_t n, int64_t nslots, int dim, int nx1,
                const int* gate = nullptr);
template <typename TD, typename TS>
void vconvert(hipStream_t st, const TS* src, TD* dst, int64_t n, const int* gate);
void vset_tol(hipStream_t st, const Red& red, double rtol);
void vset_rho(hipStream_t st, const Red& red, int sidx);
void vfill(hipStream_t st, double* dst, double value, int64_t n);
void vscale(hipStream_t st, double* v, double a, int64_t n);   // v *= a
void vmul(hipStream_t st, const double* a, const double* b, double* out, int64_t n);   // out = a o b
// y[n] = b'v_u + c v[n], the lambda row of an augmented operator, from the partials of
// b'v_u and v_u'y_u; alpha: the step length of PCG from v'y.
void vsimp_row(hipStream_t st, double* y, const double* v, int64_t n, double c, const Red& red, unsigned nblocks,
               bool alpha, const int* gate);
// dst = src, dstf = (float) src (unless null); flags[F_BAD] set unless all positive and finite
void vcopy_positive(hipStream_t st, const double* src, double* dst, float* dstf, int64_t n, const Red& red);
// Scalars, flags and *extra (may be null) into the host box, then its sequence number.
void vpublish(hipStream_t st, const Red& red, const double* extra, HostBox* box, unsigned long long seq);
void vflag_slot(hipStream_t st, const Red& red, FlagDst dst);
// Start of a PCG solve: pb = b, pu = u (clamped slots 0, flags[F_BAD] set if not
// finite), scal[S_BN2] = ||b||^2, scal[S_TOL2], scal[S_FLEX].
void vpcg_load(hipStream_t st, const double* b, const double* u, double* pb, double* pu, int64_t n, int64_t nslots,
               int dim, int nx1, const Red& red, double rtol, double flex);
void vset_omega(hipStream_t st, const Red& red, double* w, double* rho, int s_vav, int s_vdv, double omega,
                double product);
void vfill_small(hipStream_t st, double* w, int n, double value);   // n <= 64
// Bisection of the OC update (Sec. 4): x_new(lambda) = min(t / lambda, xbar) with
// sum x_new = V.  voc_init sets the bracket [0, lam_hi] and the first pass's trial
// tree; each voc_pass evaluates the sums at the OC_CAND trials of the next
// OC_LEVELS bisection levels and walks them in the order of sequential bisection
// (gated once the bracket is narrower than tau); voc_apply writes x_new at the last
// trial (blend: x_new = (blend + x_new) / 2) and its sum into scal[S_OCSUM], once
// flags[F_OCDONE] is set.  voc_bisect does all of it in one launch, where
// voc_one_workgroup(m).
bool voc_one_workgroup(int64_t m);
void voc_bisect(hipStream_t st, const double* t, int64_t m, double xbar, double V, double tau, double lam_hi,
                int max_trials, bool resume, const double* blend, double* x_new, const Red& red);
void voc_init(hipStream_t st, const Red& red, double* cand, double lam_hi);
void voc_pass(hipStream_t st, const double* t, int64_t m, double xbar, double V, double tau, double* cand,
              const Red& red);
void voc_apply(hipStream_t st, const double* t, int64_t m, double xbar, const double* blend, double* x_new,
               const Red& red);

}  // namespace ipmg
