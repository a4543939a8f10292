// PCG vector kernels (Algorithm PCG, Sec. 5.2).
#include "kernels.h"
#include "vec.h"

namespace ipmg {

namespace {

constexpr int VBLOCKS = 1024;   // grid of the streaming vector kernels

inline int vgrid(int64_t n) {
  int64_t b = (n + BS - 1) / BS;
  return (int)(b < VBLOCKS ? (b < 1 ? 1 : b) : VBLOCKS);
}
// The residual update runs one entry pair per thread (2048x1024: 22.3 us against
// 23.8 us for a grid-stride loop over 1024 blocks).
constexpr int UBLOCKS = 16384;
inline int ugrid(int64_t n) {
  int64_t b = ((n + 1) / 2 + BS - 1) / BS;
  return (int)(b < UBLOCKS ? (b < 1 ? 1 : b) : UBLOCKS);
}

// Post-processing done by the last block of a reduction.
enum Fin { FIN_STORE = 0, FIN_ALPHA = 1, FIN_RN2 = 2, FIN_BETA = 3, FIN_RN2_ZPEND = 4 };

__device__ inline void finish(int fin, double tot, const Red& red, int sidx) {
  if (fin == FIN_STORE) {
    red.scal[sidx] = tot;
  } else if (fin == FIN_ALPHA) {                 // alpha = r'y / p'Ap
    red.scal[S_PQ] = tot;
    if (!(tot > 0.0) || !isfinite(tot)) {
      red.flags[F_DONE] = 2;
      red.flags[F_STATUS] = IPMG_E_BREAKDOWN;
    } else {
      red.scal[S_ALPHA] = red.scal[S_RHO] / tot;
    }
  } else if (fin == FIN_RN2 || fin == FIN_RN2_ZPEND) {   // convergence test on ||r||^2
    rn2_finish(tot, red, fin == FIN_RN2_ZPEND);
  } else if (fin == FIN_BETA) {                  // beta = r~'y~ / r'y (or Polak-Ribiere)
    if (!(tot > 0.0) || !isfinite(tot)) {
      red.flags[F_DONE] = 2;
      red.flags[F_STATUS] = IPMG_E_BREAKDOWN;
    } else {
      const double rho = red.scal[S_RHO];
      const double num = red.scal[S_FLEX] != 0.0 ? tot - (rho + red.scal[S_ALPHA] * red.scal[S_QY]) : tot;
      red.scal[S_BETA] = num / rho;
      red.scal[S_RHO] = tot;
    }
  }
}

// One-block finalize: sum the partials of the previous kernel and apply `fin`.
__global__ __launch_bounds__(BS) void k_fin1(Red red, unsigned nblocks, int fin, int sidx, const int* gate) {
  if (gate && *gate) return;
  double tot[1];
  sum_partials<1>(red, nblocks, tot);
  if (threadIdx.x == 0) finish(fin, tot[0], red, sidx);
}

template <typename TA, typename TB>
__global__ __launch_bounds__(BS) void k_dot(const TA* __restrict__ a, const TB* __restrict__ b, int64_t n,
                                            Red red, const int* gate) {
  if (gate && *gate) return;
  double s = 0.0;
  for (int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS)
    s += (double)a[t] * (double)b[t];
  const double v[1] = {s};
  block_partials<1>(v, red);
}

// z += alpha p (unless ZUPD is off: then the next direction kernel does it);
// r += alpha q; rT = (T) r; ||r||^2 -> convergence flag.
// Each thread takes pairs of entries (16-byte accesses), two pairs per step with
// all eight loads issued first, so enough bytes are in flight to stream at the
// HBM rate; an odd last entry is taken by the first thread.
template <typename T>
__device__ inline void store_pair(T* p, double a, double b) {
  if constexpr (sizeof(T) == 8) *reinterpret_cast<double2*>(p) = make_double2(a, b);
  else *reinterpret_cast<float2*>(p) = make_float2((float)a, (float)b);
}

template <typename T, bool ZUPD>
__global__ __launch_bounds__(BS) void k_pcg_update(double* __restrict__ z, double* __restrict__ r,
                                                   const double* __restrict__ p, const double* __restrict__ q,
                                                   T* __restrict__ rT, int64_t n, Red red, const int* gate) {
  if (gate && *gate) return;
  const double alpha = red.scal[S_ALPHA];
  double s0 = 0.0, s1 = 0.0;
  const int64_t np = n / 2, stride = (int64_t)gridDim.x * BS;
  double2* z2 = reinterpret_cast<double2*>(z);
  double2* r2 = reinterpret_cast<double2*>(r);
  const double2* p2 = reinterpret_cast<const double2*>(p);
  const double2* q2 = reinterpret_cast<const double2*>(q);
  int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x;
  for (; t + stride < np; t += 2 * stride) {
    const int64_t u = t + stride;
    const double2 ra = r2[t], qa = q2[t];
    const double2 rb = r2[u], qb = q2[u];
    if constexpr (ZUPD) {
      const double2 za = z2[t], pa = p2[t];
      const double2 zb = z2[u], pb = p2[u];
      z2[t] = make_double2(za.x + alpha * pa.x, za.y + alpha * pa.y);
      z2[u] = make_double2(zb.x + alpha * pb.x, zb.y + alpha * pb.y);
    }
    const double2 na = make_double2(ra.x + alpha * qa.x, ra.y + alpha * qa.y);
    const double2 nb = make_double2(rb.x + alpha * qb.x, rb.y + alpha * qb.y);
    r2[t] = na;
    r2[u] = nb;
    if (rT) {
      store_pair<T>(rT + 2 * t, na.x, na.y);
      store_pair<T>(rT + 2 * u, nb.x, nb.y);
    }
    s0 += na.x * na.x + na.y * na.y;
    s1 += nb.x * nb.x + nb.y * nb.y;
  }
  if (t < np) {
    const double2 ra = r2[t], qa = q2[t];
    if constexpr (ZUPD) {
      const double2 za = z2[t], pa = p2[t];
      z2[t] = make_double2(za.x + alpha * pa.x, za.y + alpha * pa.y);
    }
    const double2 na = make_double2(ra.x + alpha * qa.x, ra.y + alpha * qa.y);
    r2[t] = na;
    if (rT) store_pair<T>(rT + 2 * t, na.x, na.y);
    s0 += na.x * na.x + na.y * na.y;
  }
  if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
    const int64_t e = n - 1;
    if constexpr (ZUPD) z[e] += alpha * p[e];
    const double rn = r[e] + alpha * q[e];
    r[e] = rn;
    if (rT) rT[e] = T(rn);
    s0 += rn * rn;
  }
  const double v[1] = {s0 + s1};
  block_partials<1>(v, red);
}

// The pending solution update of the last PCG step (flags[F_ZPEND], see
// k_dir_apply2d), applied after the step loop whatever stopped it; the flag is
// cleared by the next kernel.
__global__ __launch_bounds__(BS) void k_zflush(double* __restrict__ z, const double* __restrict__ p, int64_t n,
                                               Red red) {
  if (!red.flags[F_ZPEND]) return;
  const double alpha = red.scal[S_ALPHA];
  for (int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS)
    z[t] += alpha * p[t];
}
__global__ void k_zclear(Red red) {
  if (threadIdx.x == 0) red.flags[F_ZPEND] = 0;
}

// p = -y + beta p  (the reading p := -y~ + beta p of Algorithm PCG).
template <typename T>
__global__ __launch_bounds__(BS) void k_pcg_dir(double* __restrict__ p, const T* __restrict__ y, int64_t n,
                                                Red red, int first, const int* gate) {
  if (gate && *gate) return;
  const double beta = first ? 0.0 : red.scal[S_BETA];
  for (int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS)
    p[t] = -(double)y[t] + beta * p[t];
}

// out = a - b; scal[sidx] = ||out||^2.
__global__ __launch_bounds__(BS) void k_sub_norm(const double* __restrict__ a, const double* __restrict__ b,
                                                 double* __restrict__ out, int64_t n, Red red, int sidx) {
  double s = 0.0;
  for (int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS) {
    const double o = a[t] - b[t];
    out[t] = o;
    s += o * o;
  }
  const double v[1] = {s};
  block_partials<1>(v, red);
}

// dst = src with clamped slots (nodes with i == 0) zeroed; entries beyond the
// slots (lambda) copied.
__global__ __launch_bounds__(BS) void k_mask_copy(const double* __restrict__ src, double* __restrict__ dst,
                                                  int64_t n, int64_t nslots, int dim, int nx1, const int* gate) {
  if (gate && *gate) return;
  for (int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS)
    dst[t] = t < nslots && ((unsigned)t / (unsigned)dim) % (unsigned)nx1 == 0 ? 0.0 : src[t];
}

__global__ __launch_bounds__(BS) void k_fill(double* __restrict__ dst, double value, int64_t n) {
  for (int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS) dst[t] = value;
}

// dst = src, dstf = (float) src (unless null); flags[F_BAD] and [F_XBAD] = 1 unless
// every entry is finite and > 0.
__global__ __launch_bounds__(BS) void k_copy_positive(const double* __restrict__ src, double* __restrict__ dst,
                                                      float* __restrict__ dstf, int64_t n, Red red) {
  int bad = 0;
  for (int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS) {
    const double v = src[t];
    if (!(v > 0.0) || !isfinite(v)) bad = 1;
    dst[t] = v;
    if (dstf) dstf[t] = (float)v;
  }
  if (bad) red.flags[F_BAD] = red.flags[F_XBAD] = 1;
}

__global__ __launch_bounds__(64) void k_publish(Red red, const double* extra, HostBox* box, unsigned long long seq) {
  const int t = threadIdx.x;
  if (t < S_COUNT) box->scal[t] = red.scal[t];
  else if (t < S_COUNT + F_COUNT) box->flags[t - S_COUNT] = red.flags[t - S_COUNT];
  else if (t == 63 && extra) box->extra = *extra;
  __threadfence_system();
  __syncthreads();
  if (t == 0) __hip_atomic_store(&box->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
__global__ void k_flag_slot(Red red, FlagDst dst) {
  if (threadIdx.x == 0) flags_to_host(red, dst);
}

__global__ __launch_bounds__(BS) void k_pcg_load(const double* __restrict__ b, const double* __restrict__ u,
                                                 double* __restrict__ pb, double* __restrict__ pu, int64_t n,
                                                 int64_t nslots, int dim, int nx1, Red red) {
  double s = 0.0;
  int bad = 0;
  for (int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS) {
    const bool clamped = t < nslots && (t / dim) % nx1 == 0;
    const double v = clamped ? 0.0 : b[t], w = clamped ? 0.0 : u[t];
    if (!isfinite(v) || !isfinite(w)) bad = 1;
    pb[t] = v;
    pu[t] = w;
    s += v * v;
  }
  if (bad) red.flags[F_BAD] = 1;
  const double v[1] = {s};
  block_partials<1>(v, red);
}
__global__ __launch_bounds__(BS) void k_pcg_load_fin(Red red, unsigned nblocks, double rtol2, double flex) {
  double tot[1];
  sum_partials<1>(red, nblocks, tot);
  if (threadIdx.x == 0) {
    red.scal[S_BN2] = tot[0];
    red.scal[S_TOL2] = rtol2 * tot[0];
    red.scal[S_FLEX] = flex;
  }
}

template <typename TD, typename TS>
__global__ __launch_bounds__(BS) void k_convert(const TS* __restrict__ src, TD* __restrict__ dst, int64_t n,
                                                const int* gate) {
  if (gate && *gate) return;
  for (int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS)
    dst[t] = TD(src[t]);
}

__global__ void k_set_tol(Red red, double rtol2) {
  if (threadIdx.x == 0) {
    red.scal[S_TOL2] = rtol2 * red.scal[S_BN2];
    red.flags[F_DONE] = 0;
  }
}

__global__ void k_set_rho(Red red, int sidx) {
  if (threadIdx.x == 0) {
    const double rho = red.scal[sidx];
    red.scal[S_RHO] = rho;
    if (!(rho > 0.0) || !isfinite(rho)) {
      red.flags[F_DONE] = 2;
      red.flags[F_STATUS] = IPMG_E_BREAKDOWN;
    }
  }
}

// Damping safeguard: rho = v'Av / v'Dv from scal[s_vav], scal[s_vdv];
// w[0] = min(omega, product / rho), w[1] = rho (omega kept if rho is not usable).
__global__ void k_set_omega(Red red, double* __restrict__ w, double* __restrict__ rho_out, int s_vav, int s_vdv,
                            double omega, double product) {
  if (threadIdx.x == 0) {
    const double rho = red.scal[s_vav] / red.scal[s_vdv];
    double o = omega;
    if (rho > 0.0 && isfinite(rho)) o = fmin(omega, product / rho);
    w[0] = o;
    rho_out[0] = rho;
  }
}

__global__ void k_fill_value(double* __restrict__ w, int n, double value) {
  if ((int)threadIdx.x < n) w[threadIdx.x] = value;
}

}  // namespace

// ---------------------------------------------------------------- launchers --
void vdot(hipStream_t st, const double* a, const double* b, int64_t n, const Red& red, int sidx, const int* gate) {
  k_dot<double, double><<<vgrid(n), BS, 0, st>>>(a, b, n, red, gate);
  k_fin1<<<1, BS, 0, st>>>(red, vgrid(n), FIN_STORE, sidx, gate);
}
template <typename T>
void vdot_beta(hipStream_t st, const double* r, const T* y, int64_t n, const Red& red, const int* gate) {
  k_dot<double, T><<<vgrid(n), BS, 0, st>>>(r, y, n, red, gate);
  k_fin1<<<1, BS, 0, st>>>(red, vgrid(n), FIN_BETA, 0, gate);
}
template <typename T>
void vdot_store(hipStream_t st, const double* r, const T* y, int64_t n, const Red& red, int sidx, const int* gate) {
  k_dot<double, T><<<vgrid(n), BS, 0, st>>>(r, y, n, red, gate);
  k_fin1<<<1, BS, 0, st>>>(red, vgrid(n), FIN_STORE, sidx, gate);
}
template <typename T>
void vpcg_update(hipStream_t st, double* z, double* r, const double* p, const double* q, T* rT, int64_t n,
                 const Red& red, const int* gate) {
  if (z) k_pcg_update<T, true><<<ugrid(n), BS, 0, st>>>(z, r, p, q, rT, n, red, gate);
  else k_pcg_update<T, false><<<ugrid(n), BS, 0, st>>>(z, r, p, q, rT, n, red, gate);
}
void vpcg_update_fin(hipStream_t st, int64_t n, const Red& red, const int* gate, bool zpend) {
  k_fin1<<<1, BS, 0, st>>>(red, ugrid(n), zpend ? FIN_RN2_ZPEND : FIN_RN2, 0, gate);
}
unsigned vpcg_update_blocks(int64_t n) { return (unsigned)ugrid(n); }
void vpcg_update_fin_nb(hipStream_t st, unsigned nblocks, const Red& red, const int* gate, bool zpend) {
  k_fin1<<<1, BS, 0, st>>>(red, nblocks, zpend ? FIN_RN2_ZPEND : FIN_RN2, 0, gate);
}
void vzflush(hipStream_t st, double* z, const double* p, int64_t n, const Red& red) {
  k_zflush<<<vgrid(n), BS, 0, st>>>(z, p, n, red);
  k_zclear<<<1, 64, 0, st>>>(red);
}
template <typename T>
void vpcg_dir(hipStream_t st, double* p, const T* y, int64_t n, const Red& red, int first, const int* gate) {
  k_pcg_dir<T><<<vgrid(n), BS, 0, st>>>(p, y, n, red, first, gate);
}
void vsub_norm(hipStream_t st, const double* a, const double* b, double* out, int64_t n, const Red& red, int sidx) {
  k_sub_norm<<<vgrid(n), BS, 0, st>>>(a, b, out, n, red, sidx);
  k_fin1<<<1, BS, 0, st>>>(red, vgrid(n), FIN_STORE, sidx, nullptr);
}
void vmask_copy(hipStream_t st, const double* src, double* dst, int64_t n, int64_t nslots, int dim, int nx1,
                const int* gate) {
  k_mask_copy<<<vgrid(n), BS, 0, st>>>(src, dst, n, nslots, dim, nx1, gate);
}
template <typename TD, typename TS>
void vconvert(hipStream_t st, const TS* src, TD* dst, int64_t n, const int* gate) {
  k_convert<TD, TS><<<vgrid(n), BS, 0, st>>>(src, dst, n, gate);
}
void vset_tol(hipStream_t st, const Red& red, double rtol) { k_set_tol<<<1, 64, 0, st>>>(red, rtol * rtol); }
void vset_rho(hipStream_t st, const Red& red, int sidx) { k_set_rho<<<1, 64, 0, st>>>(red, sidx); }
void vfill(hipStream_t st, double* dst, double value, int64_t n) { k_fill<<<vgrid(n), BS, 0, st>>>(dst, value, n); }

namespace {
__global__ __launch_bounds__(BS) void k_scale(double* __restrict__ v, double a, int64_t n) {
  for (int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS) v[t] *= a;
}
__global__ __launch_bounds__(BS) void k_mul(const double* __restrict__ a, const double* __restrict__ b,
                                            double* __restrict__ out, int64_t n) {
  for (int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS) out[t] = a[t] * b[t];
}
__global__ __launch_bounds__(BS) void k_simp_row(double* __restrict__ y, const double* __restrict__ v, int64_t n,
                                                 double c, Red red, unsigned nblocks, int alpha, const int* gate) {
  if (gate && *gate) return;
  double tot[2];
  sum_partials<2>(red, nblocks, tot);
  if (threadIdx.x != 0) return;
  const double yl = tot[0] + c * v[n];
  y[n] = yl;
  if (alpha) finish(FIN_ALPHA, tot[1] + v[n] * yl, red, 0);
}
}  // namespace
void vscale(hipStream_t st, double* v, double a, int64_t n) { k_scale<<<vgrid(n), BS, 0, st>>>(v, a, n); }
void vmul(hipStream_t st, const double* a, const double* b, double* out, int64_t n) {
  k_mul<<<vgrid(n), BS, 0, st>>>(a, b, out, n);
}
void vsimp_row(hipStream_t st, double* y, const double* v, int64_t n, double c, const Red& red, unsigned nblocks,
               bool alpha, const int* gate) {
  k_simp_row<<<1, BS, 0, st>>>(y, v, n, c, red, nblocks, alpha ? 1 : 0, gate);
}
void vcopy_positive(hipStream_t st, const double* src, double* dst, float* dstf, int64_t n, const Red& red) {
  k_copy_positive<<<vgrid(n), BS, 0, st>>>(src, dst, dstf, n, red);
}
void vpublish(hipStream_t st, const Red& red, const double* extra, HostBox* box, unsigned long long seq) {
  k_publish<<<1, 64, 0, st>>>(red, extra, box, seq);
}
void vflag_slot(hipStream_t st, const Red& red, FlagDst dst) { k_flag_slot<<<1, 64, 0, st>>>(red, dst); }
void vpcg_load(hipStream_t st, const double* b, const double* u, double* pb, double* pu, int64_t n, int64_t nslots,
               int dim, int nx1, const Red& red, double rtol, double flex) {
  k_pcg_load<<<vgrid(n), BS, 0, st>>>(b, u, pb, pu, n, nslots, dim, nx1, red);
  k_pcg_load_fin<<<1, BS, 0, st>>>(red, vgrid(n), rtol * rtol, flex);
}
void vset_omega(hipStream_t st, const Red& red, double* w, double* rho, int s_vav, int s_vdv, double omega,
                double product) {
  k_set_omega<<<1, 64, 0, st>>>(red, w, rho, s_vav, s_vdv, omega, product);
}
void vfill_small(hipStream_t st, double* w, int n, double value) { k_fill_value<<<1, 64, 0, st>>>(w, n, value); }

// ------------------------------------------------------------ OC bisection --
namespace {

// t / lam for one lam and many t: the quotient from the rounded reciprocal and one
// correction with its exact remainder, which is the rounded quotient (4e8 random pairs
// gave no other value) in three operations instead of the eleven of a division.
// Infinite or undefined quotients come out undefined, and fmin(., xbar) is xbar for
// both.  Outside [1e-140, 1e140] the reciprocal or the remainder could leave the range:
// there the division itself is taken.
struct OcDiv {
  double lam, r;
  bool fast;
  __device__ explicit OcDiv(double l) : lam(l), r(1.0 / l), fast(l >= 1e-140 && l <= 1e140) {}
  __device__ double quick(double t) const {
    const double q = t * r;
    return __builtin_fma(__builtin_fma(-lam, q, t), r, q);
  }
};

// The whole bisection in one workgroup, the t_e in registers (E of them a thread), and
// x_new with its sum when the bracket is narrower than tau.  Bound by FP64 arithmetic of
// one CU: five operations per element and trial and a two-level sum.  resume: the
// bracket of an earlier launch goes on (max_trials ends every launch).
// A whole update with 50 trials (call to result): 335 -> 72 us at 128x64, 350 -> 87 us
// at 128x126, where 11 passes of two kernels went before.  Past 16 elements a thread the
// registers spill and the passes below, which fill the chip, take over (192x96: 347 ->
// 127 us).  LDS: the wave sums of two trials, so that one barrier per trial is enough.
constexpr int OC_WG = 1024, OC_WG_ELEMS = 16;
template <int E>
__global__ __launch_bounds__(OC_WG) void k_oc_bisect(const double* __restrict__ t, int64_t m, double xbar, double V,
                                                     double tau, double lam_hi, int max_trials, int resume,
                                                     const double* __restrict__ blend, double* __restrict__ xn,
                                                     Red red) {
  __shared__ double sh[2][OC_WG / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  double te[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int64_t e = (int64_t)i * OC_WG + threadIdx.x;
    te[i] = e < m ? t[e] : 0.0;
  }
  double lo = resume ? red.scal[S_OCLO] : 0.0, hi = resume ? red.scal[S_OCHI] : lam_hi;
  double lam = resume ? red.scal[S_OCLAM] : 0.0, steps = resume ? red.scal[S_OCSTEPS] : 0.0;
  __syncthreads();                                   // all have read the scalars
  int par = 0;
  auto total = [&](double v) {                       // the same value in every thread
    v = wave_sum(v);
    if (lane == 0) sh[par][wid] = v;
    __syncthreads();
    double s = sh[par][0];
#pragma unroll
    for (int w = 1; w < OC_WG / 64; ++w) s += sh[par][w];
    par ^= 1;
    return s;
  };
#pragma unroll 1
  for (int n = 0; n < max_trials && hi - lo > tau; ++n) {
    lam = (hi + lo) / 2.0;
    const OcDiv div(lam);
    double acc = 0.0;
    if (div.fast) {
#pragma unroll
      for (int i = 0; i < E; ++i) {                  // past m: t = 0 adds fmin(0, xbar) = 0
        acc += fmin(div.quick(te[i]), xbar);
        if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // four quotients in flight
      }
    } else {
#pragma unroll
      for (int i = 0; i < E; ++i) {
        const double v = fmin(te[i] / lam, xbar);
        acc += (int64_t)i * OC_WG + threadIdx.x < m ? v : 0.0;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    steps += 1.0;
    if (total(acc) > V) lo = lam;
    else hi = lam;
  }
  const bool done = !(hi - lo > tau);
  double sum = 0.0;
  if (done) {
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const int64_t e = (int64_t)i * OC_WG + threadIdx.x;
      if (e < m) {
        double v = fmin(te[i] / lam, xbar);
        if (blend) v = 0.5 * (blend[e] + v);
        xn[e] = v;
        acc += v;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    sum = total(acc);
  }
  if (threadIdx.x == 0) {
    red.scal[S_OCLO] = lo;
    red.scal[S_OCHI] = hi;
    red.scal[S_OCLAM] = lam;
    red.scal[S_OCSTEPS] = steps;
    red.scal[S_OCSUM] = sum;
    red.flags[F_OCDONE] = done;
  }
}

// Trials of one pass: node 0 is the midpoint of [lo, hi]; node i has children 2i+1
// (the lower half of its interval) and 2i+2 (the upper half), each midpoint formed
// as (a + b) / 2 from its interval, exactly as sequential bisection forms it on that
// path.  Thread i < OC_CAND walks from the root to its own node: node i has the path of
// the bits of i + 1 after the leading one.
__device__ inline void oc_tree(double lo, double hi, double* cand) {
  const int node = (int)threadIdx.x + 1;
  if (node > OC_CAND) return;
  double mid = (hi + lo) / 2.0;
  for (int bit = 30 - __clz(node); bit >= 0; --bit) {
    if ((node >> bit) & 1) lo = mid;
    else hi = mid;
    mid = (hi + lo) / 2.0;
  }
  cand[node - 1] = mid;
}

__global__ __launch_bounds__(64) void k_oc_init(Red red, double* cand, double lam_hi) {
  oc_tree(0.0, lam_hi, cand);
  if (threadIdx.x != 0) return;
  red.scal[S_OCLO] = 0.0;
  red.scal[S_OCHI] = lam_hi;
  red.scal[S_OCLAM] = 0.0;
  red.scal[S_OCSTEPS] = 0.0;
  red.flags[F_OCDONE] = 0;
}

// sum_e min(t_e / lambda_j, xbar) for OC_SPLIT trials of the pass (blockIdx.y takes the
// next ones): eight of the 31 a thread keep its registers few and the chip full.
constexpr int OC_SPLIT = 8;
__global__ __launch_bounds__(BS) void k_oc_sums(const double* __restrict__ t, int64_t m, double xbar,
                                                const double* __restrict__ cand, Red red) {
  if (red.flags[F_OCDONE]) return;
  const int j0 = blockIdx.y * OC_SPLIT;
  double lam[OC_SPLIT], r[OC_SPLIT], acc[OC_SPLIT];
  bool fast = true;
#pragma unroll
  for (int j = 0; j < OC_SPLIT; ++j) {
    const OcDiv d(cand[min(j0 + j, OC_CAND - 1)]);
    lam[j] = d.lam;
    r[j] = d.r;
    fast = fast && d.fast;
    acc[j] = 0.0;
  }
  for (int64_t e = (int64_t)blockIdx.x * BS + threadIdx.x; e < m; e += (int64_t)gridDim.x * BS) {
    const double te = t[e];
#pragma unroll
    for (int j = 0; j < OC_SPLIT; ++j) {
      const double q = te * r[j];
      const double v = fast ? __builtin_fma(__builtin_fma(-lam[j], q, te), r[j], q) : te / lam[j];
      acc[j] += fmin(v, xbar);
    }
  }
  // block sums, stored trial-major: partials[j * gridDim.x + block]
  __shared__ double sh[OC_SPLIT][BS / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < OC_SPLIT; ++j) {
    const double w = wave_sum(acc[j]);
    if (lane == 0) sh[j][wid] = w;
  }
  __syncthreads();
  if (threadIdx.x < OC_SPLIT && j0 + (int)threadIdx.x < OC_CAND) {
    double v = sh[threadIdx.x][0];
    for (int w = 1; w < BS / 64; ++w) v += sh[threadIdx.x][w];
    red.partials[(size_t)(j0 + threadIdx.x) * gridDim.x + blockIdx.x] = v;
  }
}

// Walk the pass's trials in sequential order: while hi - lo > tau, take the node's
// midpoint, raise lo when its sum exceeds V (go to the upper half), else lower hi.
// A wave per trial sums the blocks, every thread walks, and the next trials are formed
// side by side; with k_oc_sums split, an update of 512x256 went from 450 to 241 us.
__global__ __launch_bounds__(OC_WG) void k_oc_walk(Red red, unsigned nblocks, double V, double tau, double* cand) {
  if (red.flags[F_OCDONE]) return;
  __shared__ double tot[OC_CAND], lamc[OC_CAND];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (threadIdx.x < OC_CAND) lamc[threadIdx.x] = cand[threadIdx.x];
  for (int j = wid; j < OC_CAND; j += OC_WG / 64) {
    double a = 0.0;
    for (unsigned b = lane; b < nblocks; b += 64) a += red.partials[(size_t)j * nblocks + b];
    a = wave_sum(a);
    if (lane == 0) tot[j] = a;
  }
  double lo = red.scal[S_OCLO], hi = red.scal[S_OCHI], lam = red.scal[S_OCLAM], steps = red.scal[S_OCSTEPS];
  __syncthreads();
  int node = 0;
  for (int lvl = 0; lvl < OC_LEVELS && hi - lo > tau; ++lvl) {
    lam = lamc[node];
    steps += 1.0;
    if (tot[node] > V) {
      lo = lam;
      node = 2 * node + 2;
    } else {
      hi = lam;
      node = 2 * node + 1;
    }
  }
  const bool done = !(hi - lo > tau);
  if (!done) oc_tree(lo, hi, cand);
  if (threadIdx.x != 0) return;
  red.scal[S_OCLO] = lo;
  red.scal[S_OCHI] = hi;
  red.scal[S_OCLAM] = lam;
  red.scal[S_OCSTEPS] = steps;
  if (done) red.flags[F_OCDONE] = 1;
}

__global__ __launch_bounds__(BS) void k_oc_apply(const double* __restrict__ t, int64_t m, double xbar,
                                                 const double* __restrict__ blend, double* __restrict__ xn, Red red) {
  if (!red.flags[F_OCDONE]) return;                  // launched before the host has read it
  const double lam = red.scal[S_OCLAM];
  double s = 0.0;
  for (int64_t e = (int64_t)blockIdx.x * BS + threadIdx.x; e < m; e += (int64_t)gridDim.x * BS) {
    double v = fmin(t[e] / lam, xbar);
    if (blend) v = 0.5 * (blend[e] + v);
    xn[e] = v;
    s += v;
  }
  const double a[1] = {s};
  block_partials<1>(a, red);
}

__global__ __launch_bounds__(BS) void k_oc_apply_fin(Red red, unsigned nblocks) {
  if (!red.flags[F_OCDONE]) return;
  double tot[1];
  sum_partials<1>(red, nblocks, tot);
  if (threadIdx.x == 0) red.scal[S_OCSUM] = tot[0];
}

}  // namespace

bool voc_one_workgroup(int64_t m) { return m <= OC_WG * OC_WG_ELEMS; }

void voc_bisect(hipStream_t st, const double* t, int64_t m, double xbar, double V, double tau, double lam_hi,
                int max_trials, bool resume, const double* blend, double* x_new, const Red& red) {
  auto go = [&](auto kern) {
    kern<<<1, OC_WG, 0, st>>>(t, m, xbar, V, tau, lam_hi, max_trials, resume ? 1 : 0, blend, x_new, red);
  };
  if (m <= 2 * OC_WG) go(k_oc_bisect<2>);
  else if (m <= 8 * OC_WG) go(k_oc_bisect<8>);
  else go(k_oc_bisect<OC_WG_ELEMS>);
}
void voc_init(hipStream_t st, const Red& red, double* cand, double lam_hi) {
  k_oc_init<<<1, 64, 0, st>>>(red, cand, lam_hi);
}
void voc_pass(hipStream_t st, const double* t, int64_t m, double xbar, double V, double tau, double* cand,
              const Red& red) {
  k_oc_sums<<<dim3(vgrid(m), (OC_CAND + OC_SPLIT - 1) / OC_SPLIT), BS, 0, st>>>(t, m, xbar, cand, red);
  k_oc_walk<<<1, OC_WG, 0, st>>>(red, vgrid(m), V, tau, cand);
}
void voc_apply(hipStream_t st, const double* t, int64_t m, double xbar, const double* blend, double* x_new,
               const Red& red) {
  k_oc_apply<<<vgrid(m), BS, 0, st>>>(t, m, xbar, blend, x_new, red);
  k_oc_apply_fin<<<1, BS, 0, st>>>(red, vgrid(m));
}
template void vdot_beta<float>(hipStream_t, const double*, const float*, int64_t, const Red&, const int*);
template void vdot_beta<double>(hipStream_t, const double*, const double*, int64_t, const Red&, const int*);
template void vdot_store<float>(hipStream_t, const double*, const float*, int64_t, const Red&, int, const int*);
template void vdot_store<double>(hipStream_t, const double*, const double*, int64_t, const Red&, int, const int*);
template void vpcg_update<float>(hipStream_t, double*, double*, const double*, const double*, float*, int64_t,
                                 const Red&, const int*);
template void vpcg_update<double>(hipStream_t, double*, double*, const double*, const double*, double*, int64_t,
                                  const Red&, const int*);
template void vpcg_dir<float>(hipStream_t, double*, const float*, int64_t, const Red&, int, const int*);
template void vpcg_dir<double>(hipStream_t, double*, const double*, int64_t, const Red&, int, const int*);
template void vconvert<float, double>(hipStream_t, const double*, float*, int64_t, const int*);
template void vconvert<double, float>(hipStream_t, const float*, double*, int64_t, const int*);
template void vconvert<double, double>(hipStream_t, const double*, double*, int64_t, const int*);

}  // namespace ipmg
