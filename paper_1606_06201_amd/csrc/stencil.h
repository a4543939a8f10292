// Levels in node-stencil form: the level operator assembled into one DIM x DIM
// block per node and neighbour (3^dim neighbours), the passes of the V-cycle and
// of the damping estimate on it, and the V-cycle of all small levels in one
// workgroup.
//
// Used for the stored 3D levels, in 2D for the augmented system up to 2^18 nodes and
// for K in FP64 below the register-blocked sizes, for the damping estimates of all 2D
// levels up to 2^18 nodes, and for every level of the one-workgroup tail.  A pass over stored element matrices has to form element products and gather them
// (3D: 300 matrix entries, 24 products written and read per element, two
// launches) or to gather whole rows of 2^dim matrices per node (576 loads a node);
// the assembled rows need 243 loads a node in 3D, 36 in 2D, each read once and
// coalesced, and one launch.  The blocks are summed in FP64 and rounded once.
//
// Layout: S[(tile * NE + (c * NB + nb) * DIM + c') * 64 + lane] is the coefficient
// of component c' of neighbour nb in row c of node 64 tile + lane; a wave reads
// consecutive 64-entry rows.  Neighbours outside the grid, clamped neighbours and
// the rows of clamped nodes have zero coefficients, so every load is
// unconditional: a neighbour's index is clamped into the node range.  dinv holds
// the reciprocal diagonal per slot, 0 on clamped slots.
#pragma once
#include "kernels.h"

namespace ipmg {

template <int DIM>
struct Sten {
  static constexpr int NB = Geo<DIM>::NB;
  static constexpr int NE = NB * DIM * DIM;
  static constexpr int WAVES = DIM == 3 ? 9 : 2;   // waves per 64 nodes of a pass: (row, dz plane) or (row)
};
template <int DIM>
inline int64_t sten_size(const Dims& d) { return (d.nnodes + 63) / 64 * 64 * Sten<DIM>::NE; }

template <typename T>
struct StenLevel {
  const T* S;
  const T* dinv;
  int nn, nx1, nxy;      // nodes, nodes per row, nodes per plane
};

__device__ inline int clamp_index(int v, int n) { return min(max(v, 0), n - 1); }

// S and dinv of a level from its element matrices; one wave per (64 nodes, row c).
template <int DIM, typename T, class Op>
__global__ __launch_bounds__(64 * DIM) void k_sten_assemble(Op op, Dims d, T* __restrict__ S, T* __restrict__ dinv) {
  constexpr int NN = Geo<DIM>::NN, NB = Sten<DIM>::NB, NE = Sten<DIM>::NE;
  const int lane = threadIdx.x & 63, c = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const unsigned tile = xcd_tile().x;
  const int64_t n = (int64_t)tile * 64 + lane;
  const int i = (int)(n % d.nx1), j = (int)((n / d.nx1) % d.ny1), k = (int)(n / ((int64_t)d.nx1 * d.ny1));
  double s[NB * DIM];
#pragma unroll
  for (int t = 0; t < NB * DIM; ++t) s[t] = 0.0;
  const bool row = n < d.nnodes && i > 0;
#pragma unroll
  for (int q = 0; q < NN; ++q) {
    const int ex = q & 1, ey = (q >> 1) & 1, ez = (q >> 2) & 1;
    const int ei = i - 1 + ex, ej = j - 1 + ey, ek = k - 1 + ez;
    const bool ok = row && ei >= 0 && ei < d.nx && ej >= 0 && ej < d.ny && (DIM == 2 || (ek >= 0 && ek < d.nz));
    const int64_t e = ok ? ((int64_t)(DIM == 3 ? ek : 0) * d.ny + ej) * d.nx + ei : 0;
    const int a = loc_index(1 - ex, 1 - ey, DIM == 3 ? 1 - ez : 0);
#pragma unroll
    for (int b = 0; b < NN; ++b) {
      const int nb = nb_index<DIM>(ex + loc_x(b) - 1, ey + loc_y(b) - 1, DIM == 3 ? ez + loc_z(b) - 1 : 0);
      const bool use = ok && ei + loc_x(b) > 0;                    // a clamped column is dropped
#pragma unroll
      for (int cp = 0; cp < DIM; ++cp) {
        const double v = op.entry(e, a * DIM + c, b * DIM + cp);
        s[nb * DIM + cp] += use ? v : 0.0;
      }
    }
  }
  T* out = S + ((size_t)tile * NE + (size_t)c * NB * DIM) * 64 + lane;
#pragma unroll
  for (int t = 0; t < NB * DIM; ++t) out[(size_t)t * 64] = T(s[t]);
  double dg = 0.0;
#pragma unroll
  for (int cp = 0; cp < DIM; ++cp) dg = cp == c ? s[(NB / 2) * DIM + cp] : dg;
  if (n < d.nnodes) dinv[n * DIM + c] = row ? T(1.0 / dg) : T(0);
}

// ------------------------------------------------------------------- passes --
enum StenMode {
  ST_JACOBI2 = 0,   // out = two damped-Jacobi sweeps from zero
  ST_JACOBI = 1,    // out = v + omega D^-1 (r - A v)
  ST_RESID = 2,     // out = r - A v
  ST_BETA = 3       // ST_JACOBI and the partials of dot64'out (second partial slot)
};

// Partial dot products of a wave's lane values.
__device__ inline double lane63(double v) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63), hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
  return __hiloint2double(hi, lo);
}
template <int CTRL, int RMASK>
__device__ inline double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, RMASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, RMASK, 0xf, false);
  return v + __hiloint2double(hi, lo);
}
// Sum over the wave by row shifts and broadcasts (no LDS permutes): about a
// quarter of the latency of the shuffle form, which matters in the one-workgroup
// kernels, where a reduction follows every sweep.
__device__ inline double wave_sum_dpp(double v) {
  v = dpp_add<0x111, 0xf>(v);   // row_shr:1
  v = dpp_add<0x112, 0xf>(v);   // row_shr:2
  v = dpp_add<0x114, 0xf>(v);   // row_shr:4
  v = dpp_add<0x118, 0xf>(v);   // row_shr:8
  v = dpp_add<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v = dpp_add<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  return lane63(v);
}

// One pass over a level.  A block takes 64 nodes; in 3D wave (c, dz) sums row c
// over the neighbours of plane dz (27 coefficients and 27 values a thread, all
// loads in flight) and the first three waves add the planes; in 2D wave c takes
// row c (18 of each).  part: partial slots of this pass (b'v, then dot64'out;
// without a border dot64'out), MAX_PARTIALS apart.  lam_out: receives the lambda entry of v (LAM_SWEEP kinds).
template <int DIM, typename T, int MODE>
__global__ __launch_bounds__(64 * Sten<DIM>::WAVES) void k_sten(StenLevel<T> L, const T* __restrict__ v,
                                                                const T* __restrict__ r, T* __restrict__ out,
                                                                const double* __restrict__ omg,
                                                                const T* __restrict__ border, LamRef<T> lam,
                                                                T* lam_out, const double* __restrict__ dot64,
                                                                double* __restrict__ part, const int* gate) {
  if (gate && *gate) return;
  constexpr int NB = Sten<DIM>::NB, NE = Sten<DIM>::NE, W = Sten<DIM>::WAVES, NT = 64 * W;
  __shared__ T sh[DIM == 3 ? W : 1][64];
  __shared__ double shl[W], shr[2][DIM];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const unsigned tile = xcd_tile().x;
  const int n = (int)tile * 64 + lane;
  const int c = DIM == 3 ? w / 3 : w, seg = DIM == 3 ? w % 3 : 0;
  const T omega = T(*omg);
  const T* s = L.S + ((size_t)tile * NE + (size_t)(c * NB + seg * 9) * DIM) * 64 + lane;
  T cf[9 * DIM], x[9 * DIM], dv[MODE == ST_JACOBI2 ? 9 * DIM : 1];
#pragma unroll
  for (int t = 0; t < 9 * DIM; ++t) cf[t] = s[(size_t)t * 64];
  const int plane = DIM == 3 ? (seg - 1) * L.nxy : 0;
#pragma unroll
  for (int b = 0; b < 9; ++b) {
    const int64_t q = clamp_index(n + plane + (b / 3 - 1) * L.nx1 + (b % 3 - 1), L.nn);
    load_node<DIM, T>(MODE == ST_JACOBI2 ? r : v, q, &x[b * DIM]);
    if constexpr (MODE == ST_JACOBI2) load_node<DIM, T>(L.dinv, q, &dv[b * DIM]);
  }
  // the finishing waves' own entries
  T rr = T(0), dd = T(0), vc = T(0), bb = T(0);
  double d64 = 0.0;
  const bool fin = w < DIM, own = fin && n < L.nn;
  if (fin) {
    const size_t o = (size_t)min(n, L.nn - 1) * DIM + w;
    rr = r[o];
    if constexpr (MODE != ST_RESID) dd = L.dinv[o];
    if constexpr (MODE != ST_JACOBI2) vc = v[o];
    if (border) bb = border[o];
    if constexpr (MODE == ST_BETA) d64 = dot64[o];
  }
  const double ls = lam.nb ? wave_sum(lam_partials(lam, threadIdx.x, NT)) : 0.0;
  T acc = T(0);
#pragma unroll
  for (int t = 0; t < 9 * DIM; ++t) {
    const T xv = MODE == ST_JACOBI2 ? omega * dv[MODE == ST_JACOBI2 ? t : 0] * x[t] : x[t];
    acc += cf[t] * xv;
  }
  if constexpr (DIM == 3) sh[w][lane] = acc;
  if (lane == 0) shl[w] = ls;
  __syncthreads();
  double red0 = 0.0, red1 = 0.0;
  if (fin) {
    if constexpr (DIM == 3) acc = (sh[3 * w][lane] + sh[3 * w + 1][lane]) + sh[3 * w + 2][lane];
    T vl = T(0);
    if (border) {
      double tot = 0.0;
#pragma unroll
      for (int u = 0; u < W; ++u) tot += shl[u];
      vl = lam_value(lam, tot);
      if (lam_out && tile == 0 && threadIdx.x == 0) *lam_out = vl;
      if constexpr (MODE == ST_JACOBI2) vl = T(*omg * (double)*lam.r / lam.c);   // of the first sweep's result
      acc += bb * vl;
    }
    if constexpr (MODE == ST_JACOBI2) vc = omega * dd * rr;
    const T o = MODE == ST_RESID ? rr - acc : vc + omega * dd * (rr - acc);
    if (own) {
      out[(size_t)n * DIM + w] = o;
      red0 = (double)bb * (double)vc;
      if constexpr (MODE == ST_BETA) red1 = d64 * (double)o;
    }
  }
  if (!part) return;
  if (fin) {
    red0 = wave_sum(red0);
    if constexpr (MODE == ST_BETA) red1 = wave_sum(red1);
    if (lane == 0) {
      shr[0][w] = red0;
      shr[1][w] = red1;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = shr[0][0], b = shr[1][0];
#pragma unroll
    for (int u = 1; u < DIM; ++u) {
      a += shr[0][u];
      b += shr[1][u];
    }
    part[tile] = MODE == ST_BETA && !border ? b : a;       // the first slot, without a border
    if constexpr (MODE == ST_BETA) part[MAX_PARTIALS + tile] = b;
  }
}

// out = omega D^-1 r (the first sweep from zero alone: one pre-smoothing sweep).
template <typename T>
__global__ __launch_bounds__(BS) void k_sten_jacobi0(const T* __restrict__ dinv, const T* __restrict__ r,
                                                     T* __restrict__ out, int64_t n, const double* __restrict__ omg,
                                                     int aug, double c, const int* gate) {
  if (gate && *gate) return;
  const int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (t < n) out[t] = T(*omg) * dinv[t] * r[t];
  else if (t == n && aug) out[t] = T(*omg * (double)r[t] / c);
}

// The lambda entry of a vector whose producer left partials: one block.
template <typename T>
__global__ __launch_bounds__(BS) void k_lam_store(LamRef<T> lam, T* out, const int* gate) {
  if (gate && *gate) return;
  const T v = lam_block<T, BS>(lam);
  if (threadIdx.x == 0) *out = v;
}

// --------------------------------------------------------- damping estimate --
// Power iteration of D^-1 A and Rayleigh quotient (start vector (-1)^(i+j+k)(1+c),
// lambda 1) of several levels at a time: one launch per step for all of them, the
// norm and the lambda entry of a step's input summed by the blocks that read it
// from the previous step's partials.  (One level at a time with a one-block
// finalize per step, a set-up of the augmented system of 256 x 128 elements spent
// 430 launches on it; now 33.)
constexpr int POW_LEVELS = 8;
template <typename T>
struct PowLevel {
  StenLevel<T> L;
  const T* border;
  T* v[2];
  double* part;      // [2][3][nblk]: b'v, ||out||^2 (or v'Av), v'Dv of a step
  double* st;        // [2][2]: 1/||v||, lambda entry of a step's input
  double* w;         // results: damping, rho
  double* rho;
  int nslots, ny1;
  unsigned blk0, nblk;
};
template <typename T>
struct PowArgs {
  PowLevel<T> lv[POW_LEVELS];
  int nlev;
};
template <typename T>
__device__ inline T power_start_value(int node, int c, int nx1, int ny1) {
  const int i = node % nx1, t = node / nx1, j = t % ny1, k = t / ny1;
  return i == 0 ? T(0) : T((((i + j + k) & 1) ? -1.0 : 1.0) * (1.0 + c));
}

template <int DIM, typename T>
__global__ __launch_bounds__(64 * Sten<DIM>::WAVES) void k_sten_power(PowArgs<T> A, int step, int steps, int aug,
                                                                      double cz) {
  constexpr int NB = Sten<DIM>::NB, NE = Sten<DIM>::NE, W = Sten<DIM>::WAVES, NT = 64 * W;
  __shared__ T sh[DIM == 3 ? W : 1][64];
  __shared__ double shl[2][W], shr[3][DIM];
  int l = 0;
  while (l + 1 < A.nlev && blockIdx.x >= A.lv[l + 1].blk0) ++l;
  const PowLevel<T>& P = A.lv[l];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const unsigned tile = blockIdx.x - P.blk0;
  const int n = (int)tile * 64 + lane;
  const int c = DIM == 3 ? w / 3 : w, seg = DIM == 3 ? w % 3 : 0;
  const T* v = P.v[step & 1];
  const T* s = P.L.S + ((size_t)tile * NE + (size_t)(c * NB + seg * 9) * DIM) * 64 + lane;
  T cf[9 * DIM], x[9 * DIM];
#pragma unroll
  for (int t = 0; t < 9 * DIM; ++t) cf[t] = s[(size_t)t * 64];
  const int plane = DIM == 3 ? (seg - 1) * P.L.nxy : 0;
#pragma unroll
  for (int b = 0; b < 9; ++b) {
    const int q = clamp_index(n + plane + (b / 3 - 1) * P.L.nx1 + (b % 3 - 1), P.L.nn);
    if (step == 0) {
#pragma unroll
      for (int cp = 0; cp < DIM; ++cp) x[b * DIM + cp] = power_start_value<T>(q, cp, P.L.nx1, P.ny1);
    } else {
      load_node<DIM, T>(v, q, &x[b * DIM]);
    }
  }
  const bool fin = w < DIM, own = fin && n < P.L.nn;
  T dd = T(0), dg = T(0), vc = T(0), bb = T(0);
  if (fin) {
    const int nc = min(n, P.L.nn - 1);
    const size_t o = (size_t)nc * DIM + w;
    dd = P.L.dinv[o];
    dg = (P.L.S + ((size_t)tile * NE + (size_t)(w * NB + NB / 2) * DIM + w) * 64)[lane];
    vc = step == 0 ? power_start_value<T>(nc, w, P.L.nx1, P.ny1) : v[o];
    if (aug) bb = P.border[o];
  }
  double t0 = 0.0, t1 = 0.0;
  if (step > 0) {
    const double* pp = P.part + (size_t)((step - 1) & 1) * 3 * P.nblk;
    for (unsigned b = threadIdx.x; b < P.nblk; b += NT) {
      t0 += pp[b];
      t1 += pp[P.nblk + b];
    }
    t0 = wave_sum(t0);
    t1 = wave_sum(t1);
  }
  T acc = T(0);
#pragma unroll
  for (int t = 0; t < 9 * DIM; ++t) acc += cf[t] * x[t];
  if constexpr (DIM == 3) sh[w][lane] = acc;
  if (lane == 0) {
    shl[0][w] = t0;
    shl[1][w] = t1;
  }
  __syncthreads();
  double red[3] = {0.0, 0.0, 0.0};
  if (fin) {
    if constexpr (DIM == 3) acc = (sh[3 * w][lane] + sh[3 * w + 1][lane]) + sh[3 * w + 2][lane];
    double pin = 1.0;
    T vl = aug ? T(1) : T(0);
    if (step > 0) {
      t0 = t1 = 0.0;
#pragma unroll
      for (int u = 0; u < W; ++u) {
        t0 += shl[0][u];
        t1 += shl[1][u];
      }
      if (aug) {
        const double* sp = P.st + ((step - 1) & 1) * 2;
        const double ol = sp[0] * (t0 + cz * sp[1]) / cz;
        vl = T(ol);
        t1 += ol * ol;
      }
      pin = t1 > 0.0 ? 1.0 / sqrt(t1) : 1.0;
    }
    if (tile == 0 && threadIdx.x == 0) {
      P.st[(step & 1) * 2] = pin;
      P.st[(step & 1) * 2 + 1] = (double)vl;
    }
    if (aug) acc += bb * vl;
    if (own) {
      red[0] = (double)bb * (double)vc;
      if (step < steps) {
        const T o = T(pin * (double)(acc * dd));
        P.v[(step + 1) & 1][(size_t)n * DIM + w] = o;
        red[1] = (double)o * (double)o;
      } else {
        red[1] = (double)vc * (double)acc;
        red[2] = (double)vc * (double)dg * (double)vc;
      }
    }
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const double t = wave_sum(red[u]);
      if (lane == 0) shr[u][w] = t;
    }
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double a = shr[threadIdx.x][0];
#pragma unroll
    for (int u = 1; u < DIM; ++u) a += shr[threadIdx.x][u];
    P.part[((size_t)(step & 1) * 3 + threadIdx.x) * P.nblk + tile] = a;
  }
}

__device__ inline void store_damping(double vav, double vdv, double omega, double product, double* w, double* rho_out) {
  const double rho = vav / vdv;
  *w = rho > 0.0 && isfinite(rho) ? fmin(omega, product / rho) : omega;
  *rho_out = rho;
}

// Damping of every level from its Rayleigh partials (step `steps`): one block per level.
template <typename T>
__global__ __launch_bounds__(BS) void k_sten_power_fin(PowArgs<T> A, int steps, int aug, double cz, double omega,
                                                       double product) {
  __shared__ double sh[3][BS / 64];
  const PowLevel<T>& P = A.lv[blockIdx.x];
  const double* pp = P.part + (size_t)(steps & 1) * 3 * P.nblk;
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    double s = 0.0;
    for (unsigned b = threadIdx.x; b < P.nblk; b += BS) s += pp[(size_t)u * P.nblk + b];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) sh[u][threadIdx.x >> 6] = s;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  double t[3];
  for (int u = 0; u < 3; ++u) t[u] = (sh[u][0] + sh[u][1]) + (sh[u][2] + sh[u][3]);
  const double vl = aug ? P.st[(steps & 1) * 2 + 1] : 0.0;
  store_damping(t[1] + vl * (t[0] + cz * vl), t[2] + vl * cz * vl, omega, product, P.w, P.rho);
}

// --------------------------------------------------------------------- tail --
// V-cycle of the levels 0..top in one workgroup.  These levels hold a few thousand
// nodes in all: a launch per pass spends 4 to 5 us on less than one of work, and
// the passes of a level depend on each other, so one workgroup keeps r and two
// iterates of every level in LDS and runs a pass in 0.3 to 2 us behind a barrier.
// What bounds a pass is the instruction latency of a wave on the small levels (few
// waves have work), hence zero pads around the LDS vectors instead of index
// clamping, and what one CU reads again of the stencil on the largest.
// The coarsest solve multiplies by the stored inverse; where that is too large for
// one workgroup the tail runs as two launches (down, up) around the dense apply.
// With the finest level in the tail the launch also ends the PCG step before it
// (the direction kernel's sums, z += alpha p, r += alpha q, the stop test) and forms
// the step's ratio, so a PCG step is two launches.
constexpr int TAIL_LEVELS = 10;
constexpr int TAIL_LDS = 150 * 1024;         // bytes of level vectors
template <typename T> struct TailNT { static constexpr int value = sizeof(T) == 8 ? 512 : 1024; };   // registers

template <typename T>
struct TailLevel {
  StenLevel<T> L;
  const T* border;      // (without a border: any readable slots, the lambda entry being 0)
  T* r;                 // right-hand side in memory (the top level's; all levels when split)
  T* z;                 // iterate in memory (the top level's result; all levels when split)
  int nslots, ny1;
  float rx, ry;         // 1 / nx1, 1 / ny1
  int r_off, a_off, b_off, pad;   // LDS: r, the two iterates (level 0: the solution at a_off), zero pad after each
};
// The PCG step that the tail ends (finest level in the tail).
struct TailPcg {
  unsigned nblk = 0;    // blocks of the direction kernel (0: no step pending)
  int first = 0;
  const double* pold = nullptr;
  double *p = nullptr, *q = nullptr, *z = nullptr, *r = nullptr;
};
template <typename T>
struct TailArgs {
  TailLevel<T> lv[TAIL_LEVELS];
  int top, nu_pre, nu_post, aug;
  double cz, icz;       // corner of the augmented system (1 without one) and its reciprocal
  const double* omega;  // damping weights by level
  const T* ainv;        // A^-1 of the coarsest level, full, leading dimension ld (null: solved elsewhere)
  int ld, n0, down, up;
  TailPcg pcg;
  int r64_off;          // LDS place (in doubles) of the FP64 residual
  const double* dot64;  // PCG ratio with the result (finest level only)
  FlagDst hflags;
};

// q / d for the node counts of the tail (q < 2^16, rd = 1 / d): the quotient's
// distance from an integer is at least 0.5 / d, above the rounding of the product.
__device__ inline int tail_div(int q, float rd) { return (int)(((float)q + 0.5f) * rd); }

// A wave's tasks of a pass over a tail level: 64 nodes and all rows (2D) or one
// row (3D); task w, w + waves, ...  In 2D the coefficients, reciprocal diagonals
// and border entries of the first task are loaded once per visit of the level
// (before the transfer that precedes the passes, which hides their latency) and
// stay in registers for its passes; levels of up to 64 nodes a wave read nothing
// else.  Later tasks are streamed, and so are all tasks in 3D, where the
// coefficients of one take 81 registers.
template <int DIM, typename T>
struct TailCoef {
  static constexpr int RT = DIM == 2 ? 2 : 1, N = RT * Sten<DIM>::NB * DIM;
  T cf[N], di[RT], bo[RT];
  __device__ inline void load(const StenLevel<T>& L, const T* border, int task) {
    const int lane = threadIdx.x & 63, tile = task / (DIM / RT), c0 = task % (DIM / RT) * RT;
    const T* s = L.S + ((size_t)tile * Sten<DIM>::NE + (size_t)c0 * Sten<DIM>::NB * DIM) * 64 + lane;
#pragma unroll
    for (int t = 0; t < N; ++t) cf[t] = s[(size_t)t * 64];
    const int o = min(tile * 64 + lane, L.nn - 1) * DIM + c0;
#pragma unroll
    for (int u = 0; u < RT; ++u) {
      di[u] = L.dinv[o + u];
      bo[u] = border[o + u];
    }
  }
};
__device__ inline int tail_wave() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }
template <int DIM, typename T>
__device__ inline int tail_tasks(const StenLevel<T>& L) { return (L.nn + 63) / 64 * (DIM / TailCoef<DIM, T>::RT); }
template <int DIM, typename T>
__device__ inline void tail_load(const StenLevel<T>& L, const T* border, TailCoef<DIM, T>& K) {
  if constexpr (DIM == 2) {
    const int w = tail_wave();
    if (w < tail_tasks<DIM, T>(L)) K.load(L, border, w);
  }
}
template <int DIM, typename T, class F>
__device__ inline void tail_task(const StenLevel<T>& L, const TailCoef<DIM, T>& K, int task, const T* v, F&& f) {
  constexpr int NB = Sten<DIM>::NB, RT = TailCoef<DIM, T>::RT;
  const int tile = task / (DIM / RT), c0 = task % (DIM / RT) * RT;
  const int n = tile * 64 + (int)(threadIdx.x & 63);
  const T* vn = v + min(n, L.nn - 1) * DIM;
  T acc[RT];
#pragma unroll
  for (int u = 0; u < RT; ++u) acc[u] = T(0);
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int dz = DIM == 3 ? b / 9 - 1 : 0, dy = b / 3 % 3 - 1, dx = b % 3 - 1;
    T x[DIM];
    load_node<DIM, T>(vn + (dz * L.nxy + dy * L.nx1) * DIM, dx, x);   // outside the grid: the pad, or a zero coefficient
#pragma unroll
    for (int u = 0; u < RT; ++u)
#pragma unroll
      for (int cp = 0; cp < DIM; ++cp) acc[u] += K.cf[(u * NB + b) * DIM + cp] * x[cp];
  }
  if (n < L.nn) {
#pragma unroll
    for (int u = 0; u < RT; ++u) f(n, c0 + u, acc[u], K.di[u], K.bo[u]);
  }
}
// acc = rows of (A v) at every node of a level, v in LDS; f(node, c, sum of row c,
// reciprocal diagonal, border entry).
template <int DIM, typename T, int NT, class F>
__device__ inline void tail_rows(const StenLevel<T>& L, const T* border, const TailCoef<DIM, T>& K, const T* v, F&& f) {
  constexpr int NW = NT / 64;
  const int w = tail_wave(), nt = tail_tasks<DIM, T>(L);
  TailCoef<DIM, T> M;
  int task = w;
  if constexpr (DIM == 2) {
    if (w >= nt) return;
    task += NW;
    if (task < nt) M.load(L, border, task);
    tail_task<DIM, T>(L, K, w, v, f);
    if (task >= nt) return;
    tail_task<DIM, T>(L, M, task, v, f);
    task += NW;
  }
  for (; task < nt; task += NW) {
    M.load(L, border, task);
    tail_task<DIM, T>(L, M, task, v, f);
  }
}

// Sums over the block, in every thread; sh: two alternating rows of scratch, so
// that one barrier per call is enough.  Also the barrier of what precedes it.
template <int NT, int NV>
__device__ inline void tail_sums(double (&v)[NV], double (*sh)[3][NT / 64], int& which) {
#pragma unroll
  for (int n = 0; n < NV; ++n) {
    const double s = wave_sum_dpp(v[n]);
    if ((threadIdx.x & 63) == 0) sh[which][n][threadIdx.x >> 6] = s;
  }
  __syncthreads();
#pragma unroll
  for (int n = 0; n < NV; ++n) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) t += sh[which][n][w];
    v[n] = t;
  }
  which ^= 1;
}

// One sweep out = v + omega D^-1 (r - A v) (or the residual out = r - A v) on LDS
// vectors; lam: lambda entry of v on entry, of the result on return (aug); wc = omega / cz.
template <int DIM, typename T, int NT, bool RESID>
__device__ inline void tail_pass(const TailLevel<T>& P, const TailCoef<DIM, T>& K, const T* r, const T* v, T* out,
                                 T omega, T lr, T& lam, bool aug, double cz, double wc, double (*sh)[3][NT / 64],
                                 int& which) {
  double bd[1] = {0.0};
  tail_rows<DIM, T, NT>(P.L, P.border, K, v, [&](int n, int c, T acc, T di, T bo) {
    const int o = n * DIM + c;
    const T vc = v[o];
    acc += bo * lam;
    bd[0] += (double)bo * (double)vc;
    out[o] = RESID ? r[o] - acc : vc + omega * di * (r[o] - acc);
  });
  if (aug) {
    tail_sums<NT, 1>(bd, sh, which);
    const double row = bd[0] + cz * (double)lam;
    lam = RESID ? T((double)lr - row) : T((double)lam + wc * ((double)lr - row));
  } else {
    __syncthreads();
  }
}

// rc = P' t (the restriction's weights and order) from LDS to LDS; z1 (unless null)
// = omega D^-1 rc, the first sweep from zero.  A neighbour outside the grid is read
// in the zero pad or at a clamped node (zero); in 3D the rows above and below a
// plane's are other planes', masked.
template <int DIM, typename T, int NT>
__device__ inline void tail_restrict(const TailLevel<T>& F, const TailLevel<T>& C, const T* t, T* rc, T* z1, T omega) {
  for (int q = threadIdx.x; q < C.L.nn; q += NT) {
    const int u = tail_div(q, C.rx), I = q - u * C.L.nx1, K = DIM == 3 ? tail_div(u, C.ry) : 0, J = u - K * C.ny1;
    T d[DIM];
    if (z1) load_node<DIM, T>(C.L.dinv, q, d);
    const T* tn = t + ((2 * K * F.ny1 + 2 * J) * F.L.nx1 + 2 * I) * DIM;
    T acc[DIM];
#pragma unroll
    for (int cc = 0; cc < DIM; ++cc) acc[cc] = T(0);
#pragma unroll
    for (int dz = (DIM == 3 ? -1 : 0); dz <= (DIM == 3 ? 1 : 0); ++dz)
#pragma unroll
      for (int dy = -1; dy <= 1; ++dy) {
        const bool ok = DIM == 2 || (2 * J + dy >= 0 && 2 * J + dy < F.ny1);
#pragma unroll
        for (int dx = -1; dx <= 1; ++dx) {
          const T w = T(w1(dx) * w1(dy) * (DIM == 3 ? w1(dz) : 1.0f));
          T vv[DIM];
          load_node<DIM, T>(tn + (dz * F.L.nxy + dy * F.L.nx1) * DIM, dx, vv);
#pragma unroll
          for (int cc = 0; cc < DIM; ++cc) acc[cc] += ok ? w * vv[cc] : T(0);
        }
      }
#pragma unroll
    for (int cc = 0; cc < DIM; ++cc) acc[cc] = I > 0 ? acc[cc] : T(0);
    store_node<DIM, T>(rc, q, acc);
    if (z1) {
#pragma unroll
      for (int cc = 0; cc < DIM; ++cc) acc[cc] = omega * d[cc] * acc[cc];
      store_node<DIM, T>(z1, q, acc);
    }
  }
}

// z += P zc (the prolongation's weights and order) on LDS vectors.  The corner that
// an even coordinate does not use has weight 0; past the grid it is a pad or
// another row's entry.
template <int DIM, typename T, int NT>
__device__ inline void tail_prolong(const TailLevel<T>& F, const TailLevel<T>& C, T* z, const T* zc) {
  for (int q = threadIdx.x; q < F.L.nn; q += NT) {
    const int u = tail_div(q, F.rx), i = q - u * F.L.nx1, k = DIM == 3 ? tail_div(u, F.ry) : 0, j = u - k * F.ny1;
    const T* cn = zc + (((k >> 1) * C.ny1 + (j >> 1)) * C.L.nx1 + (i >> 1)) * DIM;
    T acc[DIM];
    load_node<DIM, T>(z, q, acc);
    const T wx[2] = {(i & 1) ? T(0.5f) : T(1), (i & 1) ? T(0.5f) : T(0)};
    const T wy[2] = {(j & 1) ? T(0.5f) : T(1), (j & 1) ? T(0.5f) : T(0)};
    const T wz[2] = {(k & 1) ? T(0.5f) : T(1), (k & 1) ? T(0.5f) : T(0)};
#pragma unroll
    for (int a = 0; a < (DIM == 3 ? 2 : 1); ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const T w = wx[e] * wy[b] * (DIM == 3 ? wz[a] : T(1));
          T vv[DIM];
          load_node<DIM, T>(cn + (a * C.L.nxy + b * C.L.nx1) * DIM, e, vv);
#pragma unroll
          for (int cc = 0; cc < DIM; ++cc) acc[cc] += w * vv[cc];
        }
#pragma unroll
    for (int cc = 0; cc < DIM; ++cc) acc[cc] = i > 0 ? acc[cc] : T(0);
    store_node<DIM, T>(z, q, acc);
  }
}

// A thread's entries of the PCG step's vectors, all loads in flight: U entries NT
// apart from `base` on (index clamped; the results past the end are not stored).
template <typename T, int NT, int U>
struct TailStep {
  double r[U], q[U], z[U], p[U];
  T d[U];
  __device__ inline void load(const TailPcg& c, const T* dinv, int base, int n) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = min(base + u * NT + (int)threadIdx.x, n - 1);
      r[u] = c.r[t];
      q[u] = c.q[t];
      z[u] = c.z[t];
      p[u] = c.p[t];
      d[u] = dinv[t];
    }
  }
};

template <int DIM, typename T>
__global__ __launch_bounds__(TailNT<T>::value) void k_tail(TailArgs<T> A, Red red, const int* gate) {
  constexpr int NT = TailNT<T>::value;
  __shared__ __align__(16) T mem[TAIL_LDS / sizeof(T)];
  __shared__ double sh[2][3][NT / 64];
  __shared__ double dsum[NT / 2], womg[TAIL_LEVELS], ratio[4];
  __shared__ T lamr[TAIL_LEVELS], lamz[TAIL_LEVELS];
  const int tid = threadIdx.x;
  const bool aug = A.aug != 0;
  int which = 0;
  // Everything the first pass needs is loaded before the gate is known.
  const TailLevel<T>& P1 = A.lv[A.top];
  TailCoef<DIM, T> K1;
  if (A.down) tail_load<DIM, T>(P1.L, P1.border, K1);
  const int stop = gate ? *gate : 0;
  if (tid <= A.top) womg[tid] = A.omega[tid];
  for (int k = 0; k <= A.top; ++k) {          // zero pads
    const TailLevel<T>& P = A.lv[k];
    for (int t = tid; t < P.pad; t += NT) {
      if (k > 0) {
        mem[P.a_off - P.pad + t] = T(0);
        mem[P.b_off - P.pad + t] = T(0);
        mem[P.b_off + P.nslots + t] = T(0);
      } else {
        mem[P.a_off + P.nslots + t] = T(0);
      }
    }
  }
  if (stop) {
    if (A.hflags.p && tid == 0) flags_to_host(red, A.hflags);
    return;
  }
  const int pre_buf = (A.nu_pre - 1) & 1;     // iterate buffer that holds z after the pre-smoothing
  if (A.down) {
    T lr = T(0);
    {
      T* r = mem + P1.r_off;
      T* z1 = mem + P1.a_off;
      const T omega = T(A.omega[A.top]);
      const int n = P1.nslots;
      if (A.pcg.nblk) {
        constexpr int U = 5;
        TailStep<T, NT, U> V;
        V.load(A.pcg, P1.L.dinv, 0, n);
        const double rho = red.scal[S_RHO], tol2 = red.scal[S_TOL2], flex = red.scal[S_FLEX];
        double v[3] = {0.0, 0.0, 0.0};
        for (unsigned b = tid; b < A.pcg.nblk; b += NT) {
          v[0] += red.partials[b];
          if (aug) v[1] += red.partials[(size_t)MAX_PARTIALS + b];
          v[2] += red.partials[2 * (size_t)MAX_PARTIALS + b];
        }
        double pl = 0.0, yl = 0.0, zl = 0.0, rl = 0.0;
        if (aug) {
          const double beta = A.pcg.first ? 0.0 : red.scal[S_BETA];
          yl = (double)P1.z[n];
          pl = -yl + (A.pcg.first ? 0.0 : beta * A.pcg.pold[n]);
          zl = A.pcg.z[n];
          rl = A.pcg.r[n];
        }
        tail_sums<NT, 3>(v, sh, which);
        const double ql = aug ? v[1] + A.cz * pl : 0.0;
        const double ptq = v[0] + pl * ql, qy = v[2] + ql * yl;
        const bool bad = !(ptq > 0.0) || !isfinite(ptq);
        const double alpha = rho / ptq;
        if (tid == 0) {
          red.scal[S_PQ] = ptq;
          red.scal[S_QY] = qy;
          if (aug) {
            A.pcg.p[n] = pl;
            A.pcg.q[n] = ql;
          }
          if (bad) {
            red.flags[F_DONE] = 2;
            red.flags[F_STATUS] = IPMG_E_BREAKDOWN;
            if (A.hflags.p) flags_to_host(red, A.hflags);
          } else {
            red.scal[S_ALPHA] = alpha;
            ratio[0] = rho;
            ratio[1] = flex != 0.0 ? rho + alpha * qy : 0.0;
          }
        }
        if (bad) return;
        double s[1] = {0.0};
        double* r64 = reinterpret_cast<double*>(mem) + A.r64_off;
        for (int base = 0; base < n; base += U * NT) {
          if (base > 0) V.load(A.pcg, P1.L.dinv, base, n);
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int t = base + u * NT + tid;
            if (t >= n) continue;
            const double rn = V.r[u] + alpha * V.q[u];
            A.pcg.z[t] = V.z[u] + alpha * V.p[u];
            A.pcg.r[t] = rn;
            s[0] = fma(rn, rn, s[0]);
            const T rt = T(rn);
            r[t] = rt;
            z1[t] = omega * V.d[u] * rt;
            if (A.r64_off >= 0) r64[t] = rn;
          }
        }
        if (aug) {
          const double rn = rl + alpha * ql;
          lr = T(rn);
          if (tid == 0) {
            A.pcg.z[n] = zl + alpha * pl;
            A.pcg.r[n] = rn;
            s[0] = fma(rn, rn, s[0]);
            ratio[2] = rn;
          }
        }
        tail_sums<NT, 1>(s, sh, which);
        const bool done = !isfinite(s[0]) || s[0] <= tol2;
        if (tid == 0) {
          rn2_finish(s[0], red, false);
          if (done && A.hflags.p) flags_to_host(red, A.hflags);
        }
        if (done) return;
      } else {
        for (int t = tid; t < n; t += NT) {
          const T rr = P1.r[t];
          r[t] = rr;
          z1[t] = omega * P1.L.dinv[t] * rr;
        }
        if (aug) lr = P1.r[n];
        __syncthreads();
      }
    }
    for (int k = A.top; k >= 1; --k) {
      const TailLevel<T>& P = A.lv[k];
      T* r = mem + P.r_off;
      T* cur = mem + P.a_off;
      T* oth = mem + P.b_off;
      const double w64 = womg[k], wc = w64 * A.icz;
      const T omega = T(w64);
      if (k < A.top) {
        const TailLevel<T>& F = A.lv[k + 1];
        tail_load<DIM, T>(P.L, P.border, K1);
        tail_restrict<DIM, T, NT>(F, P, mem + (pre_buf ? F.a_off : F.b_off), r, cur, omega);
        __syncthreads();
      }
      T lam = T(wc * (double)lr);
      for (int s = 1; s < A.nu_pre; ++s) {
        tail_pass<DIM, T, NT, false>(P, K1, r, cur, oth, omega, lr, lam, aug, A.cz, wc, sh, which);
        T* t = cur; cur = oth; oth = t;
      }
      T lt = lam;
      tail_pass<DIM, T, NT, true>(P, K1, r, cur, oth, omega, lr, lt, aug, A.cz, wc, sh, which);
      if (tid == 0) {
        lamr[k] = lr;
        lamz[k] = lam;
      }
      lr = lt;
    }
    {
      const TailLevel<T>& F = A.lv[1];
      tail_restrict<DIM, T, NT>(F, A.lv[0], mem + (pre_buf ? F.a_off : F.b_off), mem + A.lv[0].r_off, nullptr, T(0));
      if (tid == 0) lamr[0] = lr;
    }
    __syncthreads();
    if (!A.up) {                              // the coarsest solve runs elsewhere: state to memory
      for (int k = 0; k <= A.top; ++k) {
        const TailLevel<T>& P = A.lv[k];
        const T* r = mem + P.r_off;
        const T* z = mem + (pre_buf ? P.b_off : P.a_off);
        for (int t = tid; t < P.nslots; t += NT) {
          if (k < A.top || A.pcg.nblk) P.r[t] = r[t];
          if (k > 0) P.z[t] = z[t];
        }
        if (aug && tid == 0) {
          if (k < A.top || A.pcg.nblk) P.r[P.nslots] = lamr[k];
          if (k > 0) P.z[P.nslots] = lamz[k];
        }
      }
      return;
    }
    // coarsest solve z = A^-1 r: G groups of ld threads each take every G-th row of the symmetric inverse
    const TailLevel<T>& P = A.lv[0];
    const T* r = mem + P.r_off;
    T* z = mem + P.a_off;
    const int G = NT / 2 / A.ld, g = tid / A.ld, i = tid - g * A.ld;
    if (g < G) {
      double s = 0.0;
      const T* a = A.ainv + i;
      int j = g;
      for (; j + 7 * G < A.n0; j += 8 * G) {
        T av[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) av[u] = a[(size_t)(j + u * G) * A.ld];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int jj = j + u * G;
          s = fma((double)av[u], (double)(jj < P.nslots ? r[jj] : lamr[0]), s);
        }
      }
      for (; j < A.n0; j += G) s = fma((double)a[(size_t)j * A.ld], (double)(j < P.nslots ? r[j] : lamr[0]), s);
      dsum[tid] = s;
    }
    __syncthreads();
    if (tid < A.n0) {
      double t = dsum[tid];
      for (int u = 1; u < G; ++u) t += dsum[tid + u * A.ld];
      if (tid < P.nslots) z[tid] = T(t);
      else lamz[0] = T(t);
    }
    __syncthreads();
  } else {
    for (int k = 0; k <= A.top; ++k) {
      const TailLevel<T>& P = A.lv[k];
      T* r = mem + P.r_off;
      T* z = mem + (k > 0 && pre_buf ? P.b_off : P.a_off);
      for (int t = tid; t < P.nslots; t += NT) {
        r[t] = P.r[t];
        z[t] = P.z[t];
      }
      if (aug && tid == 0) {
        lamr[k] = P.r[P.nslots];
        lamz[k] = P.z[P.nslots];
      }
    }
    __syncthreads();
  }
  T lam = aug ? lamz[0] : T(0);
  const T* zc = mem + A.lv[0].a_off;
  for (int k = 1; k <= A.top; ++k) {
    const TailLevel<T>& P = A.lv[k];
    const T* r = mem + P.r_off;
    T* cur = mem + (pre_buf ? P.b_off : P.a_off);
    T* oth = mem + (pre_buf ? P.a_off : P.b_off);
    tail_load<DIM, T>(P.L, P.border, K1);
    const double w64 = womg[k], wc = w64 * A.icz;
    const T omega = T(w64);
    tail_prolong<DIM, T, NT>(P, A.lv[k - 1], cur, zc);
    if (aug) lam += lamz[k];
    const T lr = aug ? lamr[k] : T(0);
    __syncthreads();
    for (int s = 0; s < A.nu_post; ++s) {
      tail_pass<DIM, T, NT, false>(P, K1, r, cur, oth, omega, lr, lam, aug, A.cz, wc, sh, which);
      T* t = cur; cur = oth; oth = t;
    }
    zc = cur;
  }
  double s[1] = {0.0};
  const bool in_lds = A.pcg.nblk && A.r64_off >= 0;          // r of the PCG step
  const double* r64 = reinterpret_cast<const double*>(mem) + A.r64_off;
  for (int t = tid; t < P1.nslots; t += NT) {
    const T o = zc[t];
    P1.z[t] = o;
    if (A.dot64) s[0] = fma(in_lds ? r64[t] : A.dot64[t], (double)o, s[0]);
  }
  if (aug && tid == 0) P1.z[P1.nslots] = lam;
  if (A.dot64) {
    tail_sums<NT, 1>(s, sh, which);
    if (tid == 0) {
      if (aug) s[0] += (in_lds ? ratio[2] : A.dot64[P1.nslots]) * (double)lam;
      if (in_lds && s[0] > 0.0 && isfinite(s[0])) {          // finish_beta with the step's values at hand
        red.scal[S_BETA] = (s[0] - ratio[1]) / ratio[0];
        red.scal[S_RHO] = s[0];
      } else {
        finish_beta(s[0], red);
      }
    }
  }
  if (A.hflags.p && tid == 0) flags_to_host(red, A.hflags);
}

// Damping estimates of the tail's levels 1..top, one workgroup each, the vectors in LDS.
template <int DIM, typename T>
__global__ __launch_bounds__(TailNT<T>::value) void k_tail_power(TailArgs<T> A, int steps, double omega,
                                                                 double product, double* __restrict__ w,
                                                                 double* __restrict__ rho) {
  constexpr int NT = TailNT<T>::value;
  __shared__ __align__(16) T mem[TAIL_LDS / sizeof(T)];
  __shared__ double sh[2][3][NT / 64];
  int which = 0;
  const int k = 1 + (int)blockIdx.x, tid = threadIdx.x;
  const TailLevel<T>& P = A.lv[k];
  const bool aug = A.aug != 0;
  // the level's r and a slots hold the vectors' places here: pad, v, pad, o, pad
  T* v = mem + P.pad;
  T* o = v + P.nslots + P.pad;
  for (int t = tid; t < P.nslots; t += NT) v[t] = power_start_value<T>(t / DIM, t % DIM, P.L.nx1, P.ny1);
  for (int t = tid; t < P.pad; t += NT) {
    mem[t] = T(0);
    v[P.nslots + t] = T(0);
    o[P.nslots + t] = T(0);
  }
  T lam = aug ? T(1) : T(0);
  TailCoef<DIM, T> K;
  tail_load<DIM, T>(P.L, P.border, K);
  __syncthreads();
  double pin = 1.0;
  for (int it = 0; it < steps; ++it) {
    double s[2] = {0.0, 0.0};                 // ||out||^2, b'v
    tail_rows<DIM, T, NT>(P.L, P.border, K, v, [&](int n, int c, T acc, T di, T bo) {
      const int q = n * DIM + c;
      acc += bo * lam;
      s[1] += (double)bo * (double)v[q];
      const T ov = T(pin * (double)(acc * di));
      o[q] = ov;
      s[0] += (double)ov * (double)ov;
    });
    tail_sums<NT, 2>(s, sh, which);
    if (aug) {
      const double ol = pin * (s[1] + A.cz * (double)lam) / A.cz;
      lam = T(ol);
      s[0] += ol * ol;
    }
    pin = s[0] > 0.0 ? 1.0 / sqrt(s[0]) : 1.0;
    T* t = v; v = o; o = t;
  }
  double s[3] = {0.0, 0.0, 0.0};              // b'v, v'Av, v'Dv
  tail_rows<DIM, T, NT>(P.L, P.border, K, v, [&](int n, int c, T acc, T, T bo) {
    const int q = n * DIM + c;
    const double vc = (double)v[q];
    acc += bo * lam;
    s[0] += (double)bo * vc;
    s[1] += vc * (double)acc;
    const T dg = P.L.S[((size_t)(n / 64) * Sten<DIM>::NE + (c * Sten<DIM>::NB + Sten<DIM>::NB / 2) * DIM + c) * 64 + n % 64];
    s[2] += vc * (double)dg * vc;
  });
  tail_sums<NT, 3>(s, sh, which);
  const double l = (double)lam;
  if (tid == 0) store_damping(s[1] + l * (s[0] + A.cz * l), s[2] + l * A.cz * l, omega, product, w + k, rho + k);
}

}  // namespace ipmg
