// Finest 3D level: K(x) and the augmented system matrix-free, element products and
// node sums in one pass.
//
// A block owns 32 x 8 node columns and marches along z: per step every thread
// forms y_e = x_e K0 v_e (+ h_e h_e'v_e) of one element of the 33 x 9 layer, puts the
// 24 values in LDS, and every node of the plane sums its four elements below and
// four above.  Measured before as two launches (products to memory, node sums from
// it): 192 bytes an element of products written and read, 96 or 192 of h_e read;
// at 128 x 64 x 64 that was 41 us an FP32 sweep and 70 us an FP64 direction.
//
// K0 of the unit cube in the basis of the trilinear modes {1, s} x {1, t} x {1, r}: the
// sums and differences D_m of the nodal values (three butterfly stages), P = M D
// with a handful of couplings (the strain energy of the modes; cl = lambda / 16, cm =
// mu / 16, 1/3 for each linear and 1/9 for the bilinear strains), and the same
// butterflies back: about 200 operations instead of 576 multiply-adds.  The 2D
// butterflies of a node plane serve both of its layers.
// The rank-one factor h_e = s_e K0 u_e is formed from the displacements (FP64
// butterflies, then rounded to the pass's precision, as a stored h_e would be): 12
// nodal values a layer, shared, instead of 24 stored entries an element; h_e'v_e is the
// dot product of the modes.
#pragma once
#include "kernels.h"

namespace ipmg {

constexpr int F3_TX = 32, F3_TY = 8, F3_EX = F3_TX + 1, F3_EY = F3_TY + 1, F3_E = F3_EX * F3_EY;
constexpr int F3_THREADS = 320;
constexpr int F3_DIR = 100;         // mode of the PCG direction: v = -y + beta p_old, with p'q, b'p and q'y

// Modes of a component: 1, s, t, st, then the same times r.
// 2D butterfly of a plane's four nodes (counter-clockwise from (0, 0)).
template <typename T>
__device__ inline void mode_plane(const T (&v)[4][3], T (&m)[3][4]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const T a = v[0][c] + v[1][c], b = v[1][c] - v[0][c], e = v[3][c] + v[2][c], f = v[2][c] - v[3][c];
    m[c][0] = e + a;
    m[c][1] = f + b;
    m[c][2] = e - a;
    m[c][3] = f - b;
  }
}
template <typename T>
__device__ inline void mode_layer(const T (&lo)[3][4], const T (&hi)[3][4], T (&D)[3][8]) {
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      D[c][k] = hi[c][k] + lo[c][k];
      D[c][4 + k] = hi[c][k] - lo[c][k];
    }
}
// P = M D: one linear strain mode with normal strains n1, n2 (their product modes),
// the shear pair h1, h2 and the two shears that stand alone.
template <typename T>
__device__ inline void mode_linear(T cl3, T cm3, T n1, T n2, T h1, T h2, T d1, T d2, T& pn1, T& pn2, T& ph1, T& ph2,
                                   T& pd1, T& pd2) {
  const T t = cl3 * (n1 + n2), sh = cm3 * (h1 + h2), c2 = cm3 + cm3;
  pn1 += t + c2 * n1;
  pn2 += t + c2 * n2;
  ph1 += sh;
  ph2 += sh;
  pd1 += cm3 * d1;
  pd2 += cm3 * d2;
}
template <typename T>
__device__ inline void mode_stiffness(const T (&D)[3][8], T cl, T cm, T (&P)[3][8]) {
  constexpr int S = 1, Q = 2, SQ = 3, R = 4, SR = 5, QR = 6, A = 7;    // s, t, st, r, sr, tr, str
  const T cm2 = cm + cm, t = cl * (D[0][S] + D[1][Q] + D[2][R]);
#pragma unroll
  for (int c = 0; c < 3; ++c) P[c][0] = P[c][SQ] = P[c][SR] = P[c][QR] = T(0);
  P[0][S] = t + cm2 * D[0][S];
  P[1][Q] = t + cm2 * D[1][Q];
  P[2][R] = t + cm2 * D[2][R];
  P[0][Q] = P[1][S] = cm * (D[0][Q] + D[1][S]);
  P[0][R] = P[2][S] = cm * (D[0][R] + D[2][S]);
  P[1][R] = P[2][Q] = cm * (D[1][R] + D[2][Q]);
  const T cl3 = cl * T(1.0 / 3.0), cm3 = cm * T(1.0 / 3.0);
  mode_linear(cl3, cm3, D[0][SQ], D[2][QR], D[0][QR], D[2][SQ], D[1][SQ], D[1][QR], P[0][SQ], P[2][QR], P[0][QR],
              P[2][SQ], P[1][SQ], P[1][QR]);
  mode_linear(cl3, cm3, D[1][SQ], D[2][SR], D[1][SR], D[2][SQ], D[0][SQ], D[0][SR], P[1][SQ], P[2][SR], P[1][SR],
              P[2][SQ], P[0][SQ], P[0][SR]);
  mode_linear(cl3, cm3, D[0][SR], D[1][QR], D[0][QR], D[1][SR], D[2][SR], D[2][QR], P[0][SR], P[1][QR], P[0][QR],
              P[1][SR], P[2][SR], P[2][QR]);
  const T c9 = (cl + T(4) * cm) * T(1.0 / 9.0);
#pragma unroll
  for (int c = 0; c < 3; ++c) P[c][A] = c9 * D[c][A];
}
// Nodal values of a plane from its four modes.
template <typename T>
__device__ inline void mode_nodes(const T (&m)[4], T (&f)[4]) {
  const T a = m[0] - m[2], b = m[1] - m[3], e = m[0] + m[2], g = m[1] + m[3];
  f[0] = a - b;
  f[1] = a + b;
  f[2] = e + g;
  f[3] = e - g;
}

template <typename T>
struct Fine3 {
  const T* x;          // densities
  const T* dgn;        // diagonal per slot
  const double* u;     // augmented system: displacements (0 on clamped slots) and s_e of h_e = s_e K0 u_e
  const double* s;
  double cl, cm;       // lambda / 16, mu / 16
};
// The PCG direction's vectors (F3_DIR).
template <typename TY>
struct Dir3 {
  const TY* y = nullptr;
  const double* pold = nullptr;
  double* p = nullptr;
  int first = 0;
};

// MODE: a LevelMode (M_JACOBI2: the two sweeps from zero, v = omega D^-1 r formed on
// the fly; its lambda entry is stored to vlam) or F3_DIR.  TZ: node planes a block.
// Column i = 0 is clamped: the tiles start at i = 1 and the first one stores its zeros.
template <typename T, bool Z, int MODE, typename TY>
__global__ __launch_bounds__(F3_THREADS) void k_fine3(Fine3<T> op, Dims d, int TZ, const T* __restrict__ v,
                                                      const T* __restrict__ r, T* __restrict__ out,
                                                      const double* __restrict__ omg, Aug<T> aug, Red red,
                                                      int sidx_in, const double* __restrict__ dot64, T* vlam,
                                                      Dir3<TY> dir, const int* gate) {
  if (gate && *gate) return;
  constexpr bool DIR = MODE == F3_DIR;
  constexpr bool DIAG = !DIR && MODE != M_APPLY && MODE != M_RESID;
  // FP32: two layers, so that one barrier a step is enough; FP64: one (two would
  // leave a CU one block)
  constexpr int NY = sizeof(T) == 4 ? 2 : 1;
  __shared__ T YY[NY][24][F3_E];
  const int tid = threadIdx.x;
  const T omega = omg ? T(*omg) : T(0);
  const T cl = T(op.cl), cm = T(op.cm);
  double pin = 1.0;
  if constexpr (MODE == M_POWER) {
    if (sidx_in >= 0) {
      const double s = red.scal[sidx_in];
      pin = s > 0.0 ? 1.0 / sqrt(s) : 1.0;
    }
  }
  double beta = 0.0;
  if constexpr (DIR) beta = dir.first ? 0.0 : red.scal[S_BETA];
  T vl = T(0);                                     // lambda entry of v
  if (aug.b) {
    if constexpr (DIR) vl = -(double)dir.y[aug.n] + (dir.first ? 0.0 : beta * dir.pold[aug.n]);
    else if constexpr (MODE == M_JACOBI2) vl = T((double)omega * (double)r[aug.n] / aug.c);
    else vl = v[aug.n];
  }
  const Tile tl = xcd_tile();
  if constexpr (MODE == M_JACOBI2) {
    if (aug.b && tl.x == 0 && tl.y == 0 && tl.z == 0 && tid == 0) vlam[aug.n] = vl;
  }
  const int i0 = 1 + (int)tl.x * F3_TX, j0 = (int)tl.y * F3_TY, k0 = (int)tl.z * TZ, k1 = min(k0 + TZ, d.nz1);
  // the thread's element column
  const int ex = tid % F3_EX, ey = tid / F3_EX, ei = i0 - 1 + ex, ej = j0 - 1 + ey;
  const bool eok = tid < F3_E && ei < d.nx && ej >= 0 && ej < d.ny;
  const int ia = min(ei, d.nx), ib = min(ei + 1, d.nx), ja = min(max(ej, 0), d.ny), jb = min(max(ej + 1, 0), d.ny);
  const int nq[4] = {ja * d.nx1 + ia, ja * d.nx1 + ib, jb * d.nx1 + ib, jb * d.nx1 + ia};
  const int plane = d.nx1 * d.ny1;
  const int eq = min(max(ej, 0), d.ny - 1) * d.nx + min(ei, d.nx - 1);
  // and its node column
  const int tx = tid % F3_TX, ty = tid / F3_TX, i = i0 + tx, j = j0 + ty;
  const bool nok = tid < F3_TX * F3_TY && i < d.nx1 && j < d.ny1;
  const int nc = min(j, d.ny) * d.nx1 + min(i, d.nx);
  const int y00 = ty * F3_EX + tx;                 // LDS place of element (i-1, j-1) of the layer

  auto value = [&](int64_t o) -> T {               // v at slot o
    if constexpr (DIR) return -(double)dir.y[o] + beta * dir.pold[o];
    else if constexpr (MODE == M_JACOBI2) return omega * r[o] * (op.dgn[o] != T(0) ? recip(op.dgn[o]) : T(0));
    else return v[o];
  };
  auto load_plane = [&](int k, T (&a)[4][3]) {
    const int64_t b = (int64_t)min(max(k, 0), d.nz) * plane;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int c = 0; c < 3; ++c) a[q][c] = value(3 * (b + nq[q]) + c);
  };
  auto load_u = [&](int k, double (&a)[4][3]) {
    const int64_t b = (int64_t)min(max(k, 0), d.nz) * plane;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int c = 0; c < 3; ++c) a[q][c] = op.u[3 * (b + nq[q]) + c];
  };
  auto layer_at = [&](int k) { return (int64_t)min(max(k, 0), d.nz - 1) * d.nx * d.ny + eq; };

  T vn[4][3], vlo[3][4], vhi[3][4];
  double un[Z ? 4 : 1][3], ulo[3][4], uhi[3][4];
  load_plane(k0 - 1, vn);
  mode_plane(vn, vlo);
  if constexpr (Z) {
    load_u(k0 - 1, un);
    mode_plane(un, ulo);
  }
  load_plane(k0, vn);
  if constexpr (Z) load_u(k0, un);
  T xe = op.x[layer_at(k0 - 1)];
  double se = 0.0;
  if constexpr (Z) se = op.s[layer_at(k0 - 1)];
  T carry[3] = {T(0), T(0), T(0)};
  double red0 = 0.0, red1 = 0.0, bdot = 0.0;       // F3_DIR: q'y, p'q, b'p
  for (int ek = k0 - 1; ek < k1; ++ek) {
    // entries of the node of plane ek, used after the barrier
    const int64_t qn = (int64_t)max(ek, 0) * plane + nc, sl = 3 * qn;
    T rr[3] = {T(0), T(0), T(0)}, dg[3] = {T(1), T(1), T(1)}, vc[3], bb[3] = {T(0), T(0), T(0)}, yc[3] = {T(0), T(0), T(0)};
    double d64[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if constexpr (!DIR && MODE != M_APPLY && MODE != M_POWER && MODE != M_RAYLEIGH) rr[c] = r[sl + c];
      if constexpr (DIAG) dg[c] = op.dgn[sl + c];
      vc[c] = value(sl + c);
      if (aug.b) bb[c] = aug.b[sl + c];
      if constexpr (DIR) yc[c] = (T)dir.y[sl + c];
      if constexpr (MODE == M_JACOBI_BETA) d64[c] = dot64[sl + c];
    }
    mode_plane(vn, vhi);
    if constexpr (Z) mode_plane(un, uhi);
    T(&Y)[24][F3_E] = YY[NY == 2 ? ek & 1 : 0];
    {
      const bool ok = eok && ek >= 0 && ek < d.nz;
      T D[3][8], P[3][8];
      mode_layer(vlo, vhi, D);
      mode_stiffness(D, cl, cm, P);
      const T xk = ok ? xe : T(0);
      if constexpr (Z) {
        double U[3][8], H[3][8];
        mode_layer(ulo, uhi, U);
        mode_stiffness(U, op.cl, op.cm, H);
        const double sk = ok ? se : 0.0;
        T hv = T(0), h[3][8];
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
          for (int m = 1; m < 8; ++m) {
            h[c][m] = T(sk * H[c][m]);
            hv += h[c][m] * D[c][m];
          }
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
          for (int m = 1; m < 8; ++m) P[c][m] = xk * P[c][m] + h[c][m] * hv;
      } else {
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
          for (int m = 1; m < 8; ++m) P[c][m] *= xk;
      }
      if (tid < F3_E) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const T lo[4] = {-P[c][4], P[c][1] - P[c][5], P[c][2] - P[c][6], P[c][3] - P[c][7]};
          const T hi[4] = {P[c][4], P[c][1] + P[c][5], P[c][2] + P[c][6], P[c][3] + P[c][7]};
          T f[4];
          mode_nodes(lo, f);
#pragma unroll
          for (int a = 0; a < 4; ++a) Y[a * 3 + c][tid] = f[a];
          mode_nodes(hi, f);
#pragma unroll
          for (int a = 0; a < 4; ++a) Y[(4 + a) * 3 + c][tid] = f[a];
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        vlo[c][m] = vhi[c][m];
        if constexpr (Z) ulo[c][m] = uhi[c][m];
      }
    // the next layer's loads are in flight through the node part
    load_plane(ek + 2, vn);
    if constexpr (Z) load_u(ek + 2, un);
    xe = op.x[layer_at(ek + 1)];
    if constexpr (Z) se = op.s[layer_at(ek + 1)];
    __syncthreads();
    if (tid < F3_TX * F3_TY) {
      T acc[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        // elements (i-1, j-1), (i, j-1), (i, j), (i-1, j): the node is their corner 2, 3, 0, 1
        const T lo = (Y[6 + c][y00] + Y[9 + c][y00 + 1]) + (Y[c][y00 + F3_EX + 1] + Y[3 + c][y00 + F3_EX]);
        const T hi = (Y[18 + c][y00] + Y[21 + c][y00 + 1]) + (Y[12 + c][y00 + F3_EX + 1] + Y[15 + c][y00 + F3_EX]);
        acc[c] = carry[c] + lo;
        carry[c] = hi;
      }
      if (ek >= k0 && nok) {
        if constexpr (DIR) {
          double pc[3], o[3];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            pc[c] = vc[c];
            o[c] = acc[c] + bb[c] * vl;
            bdot += bb[c] * pc[c];
            red1 += pc[c] * o[c];
            red0 += o[c] * yc[c];
          }
          store_node<3, double>(dir.p, qn, pc);
          store_node<3, double>(out, qn, o);
        } else {
          level_node_finish_vals<3, T, MODE>(qn, acc, dg, vc, rr, out, omega, aug.b != nullptr, bb, vl, pin, d64, bdot,
                                             red0, red1);
        }
      }
      if (ek >= k0 && i == 1 && j < d.ny1) {       // the clamped node of the row
        const T z[3] = {T(0), T(0), T(0)};
        if constexpr (MODE != M_RAYLEIGH) store_node<3, T>(out, qn - 1, z);
        if constexpr (DIR) store_node<3, double>(dir.p, qn - 1, z);
      }
    }
    if constexpr (NY == 1) __syncthreads();
  }
  constexpr bool NEED = MODE == M_POWER || MODE == M_RAYLEIGH || MODE == M_JACOBI_BETA;
  if (DIR || aug.b || NEED) {
    const double vals[3] = {DIR ? red1 : bdot, DIR ? bdot : red0, DIR ? red0 : red1};
    const double level_vals[3] = {bdot, red0, red1}, plain[3] = {red0, red1, 0.0};
    if constexpr (DIR) block_partials<3, false, F3_THREADS>(vals, red);
    else if (aug.b) block_partials<3, false, F3_THREADS>(level_vals, red);
    else block_partials<3, false, F3_THREADS>(plain, red);
  }
}

}  // namespace ipmg
