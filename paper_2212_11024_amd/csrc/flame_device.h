// Device-side lattice tables, storage encodings and per-node arithmetic of the coupled
// Hall-MHD lattice-Boltzmann step (paper Sec. 3.1-3.2, App. A-B).
//
// Populations are carried as deviations from the rest state of the run,
//   df_i = f_i - f_rest_i,  f_rest = f^mhd(0)(1, 0, b0);   dg_ia = g_ia - W_i b0_a,
// so that FP32/FP16 storage keeps its precision for the small departures that carry the
// physics. All per-node arithmetic below is written in terms of these deviations.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// Per-node arithmetic is host-and-device so the same code can be exercised on the CPU.
#define FLAME_HD __host__ __device__ __forceinline__

namespace flame {

// ------------------------------------------------------------------ lattice tables
// D3Q27 velocities in the order of the paper's App. A listing.
__host__ __device__ constexpr int cq(int i, int a) {
  constexpr int8_t t[27][3] = {
      {0, 0, 0},   {-1, 0, 0},  {0, -1, 0},  {0, 0, -1}, {-1, -1, 0}, {-1, 1, 0},  {-1, 0, -1},
      {-1, 0, 1},  {0, -1, -1}, {0, -1, 1},  {-1, -1, -1}, {-1, -1, 1}, {-1, 1, -1}, {-1, 1, 1},
      {1, 0, 0},   {0, 1, 0},   {0, 0, 1},   {1, 1, 0},  {1, -1, 0},  {1, 0, 1},   {1, 0, -1},
      {0, 1, 1},   {0, 1, -1},  {1, 1, 1},   {1, 1, -1}, {1, -1, 1},  {1, -1, -1}};
  return t[i][a];
}
// In the App. A listing the opposite of direction i (1 <= i <= 13) is i + 13.
__host__ __device__ constexpr int oppq(int i) { return i == 0 ? 0 : (i <= 13 ? i + 13 : i - 13); }
// Index of the D3Q27 direction (x, y, z) in the App. A order.
__host__ __device__ constexpr int qindex(int x, int y, int z) {
  int k = 0;
  for (int i = 0; i < 27; ++i)
    if (cq(i, 0) == x && cq(i, 1) == y && cq(i, 2) == z) k = i;
  return k;
}
__host__ __device__ constexpr int speed2q(int i) {
  return cq(i, 0) * cq(i, 0) + cq(i, 1) * cq(i, 1) + cq(i, 2) * cq(i, 2);
}
// Weights by speed class (Sec. 3.1): 8/27, 2/27, 1/54, 1/216.
__host__ __device__ constexpr double wq(int i) {
  return speed2q(i) == 0 ? 8.0 / 27.0
       : speed2q(i) == 1 ? 2.0 / 27.0
       : speed2q(i) == 2 ? 1.0 / 54.0
                          : 1.0 / 216.0;
}
// D3Q7: rest, -x, -y, -z, +x, +y, +z. Weights 1/4 (rest), 1/8 (faces); C^2 = 1/4.
__host__ __device__ constexpr int xim(int i, int a) {
  return i == 0 ? 0 : (i <= 3 ? (a == i - 1 ? -1 : 0) : (a == i - 4 ? 1 : 0));
}
__host__ __device__ constexpr int oppm(int i) { return i == 0 ? 0 : (i <= 3 ? i + 3 : i - 3); }
__host__ __device__ constexpr double wm(int i) { return i == 0 ? 0.25 : 0.125; }

constexpr int kQ = 27;
constexpr int kM = 21;   // 7 directions x 3 components, index i * 3 + component

// ------------------------------------------------------------------ storage encodings
// Power-of-two scales applied to stored deviations (exact in every format); only FP16
// needs them, to keep deviations of magnitude ~ w_i |u| clear of the subnormal range.
template <typename S>
struct Enc;

template <>
struct Enc<double> {
  using R = double;
  static __host__ __device__ constexpr double fscale(int) { return 1.0; }
  static __host__ __device__ constexpr double mscale(int) { return 1.0; }
  static __device__ __forceinline__ double dec(double v, double) { return v; }
  static __device__ __forceinline__ double enc(double v, double) { return v; }
};

template <>
struct Enc<float> {
  using R = float;
  static __host__ __device__ constexpr double fscale(int) { return 1.0; }
  static __host__ __device__ constexpr double mscale(int) { return 1.0; }
  static __device__ __forceinline__ float dec(float v, float) { return v; }
  static __device__ __forceinline__ float enc(float v, float) { return v; }
};

template <>
struct Enc<_Float16> {
  using R = float;
  static __host__ __device__ constexpr double fscale(int i) {
    return speed2q(i) == 0 ? 4.0 : speed2q(i) == 1 ? 16.0 : speed2q(i) == 2 ? 64.0 : 256.0;
  }
  static __host__ __device__ constexpr double mscale(int i) { return i == 0 ? 4.0 : 8.0; }
  static __device__ __forceinline__ float dec(_Float16 v, float inv_scale) {
    return static_cast<float>(v) * inv_scale;
  }
  static __device__ __forceinline__ _Float16 enc(float v, float scale) {
    return static_cast<_Float16>(v * scale);
  }
};

// ------------------------------------------------------------------ run constants
template <typename R>
struct PhysConst {
  R omega;       // fluid relaxation rate, 1/omega = 3 nu + 1/2
  R omega_b;     // magnetic relaxation rate, 1/omega_B = 4 eta + 1/2
  R alpha;       // Hall coefficient alpha_H (= d_i in cells)
  R b0[3];       // background field
};

// ------------------------------------------------------------------ per-node arithmetic
// Fluid moments of the deviations: d rho = sum df, j = sum df c, S2 = sum df c c.
template <typename R>
struct FluidMoments {
  R drho, jx, jy, jz, sxx, syy, szz, sxy, sxz, syz;
};

// Summed axis by axis (z, then y, then x): 66 additions instead of the 161 of ten separate sums.
template <typename R>
FLAME_HD FluidMoments<R> fluid_moments(const R (&f)[kQ]) {
  FluidMoments<R> m{};
  R t[3][3], d[3][3], s[3][3];   // per (c_x, c_y): sum over c_z, sum of c_z f, sum of c_z^2 f
#pragma unroll
  for (int X = 0; X < 3; ++X)
#pragma unroll
    for (int Y = 0; Y < 3; ++Y) {
      const R lo = f[qindex(X - 1, Y - 1, -1)], hi = f[qindex(X - 1, Y - 1, 1)];
      s[X][Y] = hi + lo;
      d[X][Y] = hi - lo;
      t[X][Y] = s[X][Y] + f[qindex(X - 1, Y - 1, 0)];
    }
  R t0[3], t1[3], t2[3], d0[3], d1[3], s0[3];   // per c_x: the same over c_y
#pragma unroll
  for (int X = 0; X < 3; ++X) {
    t2[X] = t[X][2] + t[X][0];
    t1[X] = t[X][2] - t[X][0];
    t0[X] = t2[X] + t[X][1];
    d1[X] = d[X][2] - d[X][0];
    d0[X] = d[X][2] + d[X][0] + d[X][1];
    s0[X] = s[X][2] + s[X][0] + s[X][1];
  }
  m.sxx = t0[2] + t0[0];
  m.jx = t0[2] - t0[0];
  m.drho = m.sxx + t0[1];
  m.jy = t1[2] + t1[0] + t1[1];
  m.sxy = t1[2] - t1[0];
  m.syy = t2[2] + t2[0] + t2[1];
  m.jz = d0[2] + d0[0] + d0[1];
  m.sxz = d0[2] - d0[0];
  m.syz = d1[2] + d1[0] + d1[1];
  m.szz = s0[2] + s0[0] + s0[1];
  return m;
}

// Field fluctuation b = sum dg (the rest part sums to b0) and Lambda_ab = sum_i xi_ia g_ib,
// which for D3Q7 is the difference of the +a and -a populations (the rest part cancels).
template <typename R>
FLAME_HD void magnetic_moments(const R (&g)[kM], R (&b)[3], R (&lam)[3][3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    R s = g[a];
#pragma unroll
    for (int i = 1; i < 7; ++i) s += g[i * 3 + a];
    b[a] = s;
  }
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c) lam[a][c] = g[(4 + a) * 3 + c] - g[(1 + a) * 3 + c];
}

// Field fluctuation component c of a node from its magnetic populations, with the source
// half-shift; one fixed summation order everywhere so a node's b is bitwise the same
// whichever thread computes it.
template <typename R>
FLAME_HD R b_component(const R (&g)[kM], int c, R half_src) {
  R s = g[c];
#pragma unroll
  for (int i = 1; i < 7; ++i) s += g[i * 3 + c];
  return s + half_src;
}

// J from the magnetic first moment (Sec. 3.2): (I + 2 alpha w_B / C^2 M(B)) J = -(w_B/C^2) J0,
// M(B) J = J x B, J0 = eps:Lambda - 2 U x B. Written as J + k (J x B) = r, whose solution is
// J = (r - k r x B + k^2 (r . B) B) / (1 + k^2 |B|^2), with k = 8 alpha w_B and r = -4 w_B J0.
template <typename R>
FLAME_HD void current_from_moments(const R (&lam)[3][3], const R (&U)[3],
                                                     const R (&B)[3], R alpha, R omega_b,
                                                     R (&J)[3]) {
  const R j0x = lam[1][2] - lam[2][1] - R(2) * (U[1] * B[2] - U[2] * B[1]);
  const R j0y = lam[2][0] - lam[0][2] - R(2) * (U[2] * B[0] - U[0] * B[2]);
  const R j0z = lam[0][1] - lam[1][0] - R(2) * (U[0] * B[1] - U[1] * B[0]);
  const R s = R(-4) * omega_b;
  const R rx = s * j0x, ry = s * j0y, rz = s * j0z;
  const R k = R(8) * alpha * omega_b;
  const R rbx = ry * B[2] - rz * B[1], rby = rz * B[0] - rx * B[2], rbz = rx * B[1] - ry * B[0];
  const R rdb = rx * B[0] + ry * B[1] + rz * B[2];
  const R k2 = k * k;
  const R inv = R(1) / (R(1) + k2 * (B[0] * B[0] + B[1] * B[1] + B[2] * B[2]));
  J[0] = (rx - k * rbx + k2 * rdb * B[0]) * inv;
  J[1] = (ry - k * rby + k2 * rdb * B[1]) * inv;
  J[2] = (rz - k * rbz + k2 * rdb * B[2]) * inv;
}

// 1-D factors on c in {-1, 0, +1} (index c + 1):
//  e(c) = phi(c; u) / w1(c) - 1, phi the D1Q3 equilibrium (its 3-D product is the
//        sixth-order Hermite f^(0) of App. A): e(0) = -3u^2/2, e(+-1) = 3u^2 +- 3u;
//  h_p(c): central moments about u equal to delta_{p,q} for q = 0, 1, 2.
template <typename R>
struct Axis {
  R e[3], h0[3], h1[3], h2[3];
  FLAME_HD explicit Axis(R u) {
    const R u2 = u * u;
    e[0] = R(3) * (u2 - u); e[1] = R(-1.5) * u2; e[2] = R(3) * (u2 + u);
    h0[0] = R(0.5) * (u2 - u); h0[1] = R(1) - u2; h0[2] = R(0.5) * (u2 + u);
    h1[0] = u - R(0.5); h1[1] = R(-2) * u; h1[2] = u + R(0.5);
    h2[0] = R(0.5); h2[1] = R(-1); h2[2] = R(0.5);
  }
};

// ------------------------------------------------------------------ separable D3Q27 transforms
// A D3Q27 distribution as a tensor product: along one axis a distribution on c = -1, 0, +1 with
// moments m0, m1, m2 has the Hermite coefficients (m0, m1, a2 = m2 - m0 / 3), and
//   t = m0 / 6 + a2 / 2,  f(+-1) = t +- m1 / 2,  f(0) = m0 - 2 t.
// Stored per axis as (m0, m1 / 2, a2 / 2), index p * 9 + q * 3 + r for the orders along x, y, z.
// In this basis the equilibrium rho phi(u_x) phi(u_y) phi(u_z) has the coefficients
// rho u_x^p u_y^q u_z^r (so its deviation from rest is formed without cancellation), the Maxwell
// stress enters the six second-order coefficients only, and a distribution given by its
// coefficients about u is moved to the lattice frame by the shift below. One shift (three passes of
// 9 lines) and one back-transform (the same) replace 27 separate polynomial evaluations: about 250
// instead of 700 arithmetic operations per node, and about 1000 instead of 4500 in the reverse pass.
FLAME_HD constexpr int tidx(int p, int q, int r) { return p * 9 + q * 3 + r; }

// Line l (0..8) of axis A: its three entries are base, base + step, base + 2 step.
template <int A>
FLAME_HD constexpr int line_step() { return A == 0 ? 9 : A == 1 ? 3 : 1; }
template <int A>
FLAME_HD constexpr int line_base(int l) {
  return A == 0 ? l : A == 1 ? (l / 3) * 9 + l % 3 : l * 3;
}

// Coefficients about u -> coefficients about 0 along axis A:
// m1 = c1 + u c0, a2 = c2 + 2 u c1 + u^2 c0.
template <int A, typename R>
FLAME_HD void shift_axis(R (&a)[kQ], R u) {
  const R hu = R(0.5) * u, u2 = u + u, huu = hu * u;
  constexpr int s = line_step<A>();
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int i = line_base<A>(l);
    a[i + 2 * s] += u2 * a[i + s] + huu * a[i];
    a[i + s] += hu * a[i];
  }
}
// Its transpose.
template <int A, typename R>
FLAME_HD void shift_axis_t(R (&a)[kQ], R u) {
  const R hu = R(0.5) * u, u2 = u + u, huu = hu * u;
  constexpr int s = line_step<A>();
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int i = line_base<A>(l);
    a[i] += hu * a[i + s] + huu * a[i + 2 * s];
    a[i + s] += u2 * a[i + 2 * s];
  }
}
// Coefficients -> populations along axis A (entries become c = -1, 0, +1).
template <int A, typename R>
FLAME_HD void populate_axis(R (&a)[kQ]) {
  constexpr int s = line_step<A>();
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int i = line_base<A>(l);
    const R m0 = a[i], m1 = a[i + s], a2 = a[i + 2 * s];
    const R t = m0 * R(1.0 / 6.0) + a2;
    a[i] = t - m1;
    a[i + s] = m0 - (t + t);   // not 2/3 m0 - 2 a2: the three then sum to m0 without a rounded constant's bias
    a[i + 2 * s] = t + m1;
  }
}
// Its transpose.
template <int A, typename R>
FLAME_HD void populate_axis_t(R (&a)[kQ]) {
  constexpr int s = line_step<A>();
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int i = line_base<A>(l);
    const R lo = a[i], mid = a[i + s], hi = a[i + 2 * s];
    const R lt = (hi + lo) - (mid + mid);
    a[i] = mid + lt * R(1.0 / 6.0);
    a[i + s] = hi - lo;
    a[i + 2 * s] = lt;
  }
}

// Coefficients about U of a fluid distribution with density coefficient rho, deviatoric central
// second moments Q (xx, yy, zz, xy, xz, yz) and first central moments fh; every other central
// moment is that of the equilibrium. (A unit central moment along some axes is the distribution
// h0 = (1, 0, -1/3) along the others; the c_220 type entries use tr Q = 0.)
template <typename R>
FLAME_HD void central_coefficients(R rho, const R (&Q)[6], const R (&fh)[3], R (&c)[kQ]) {
  c[tidx(0, 0, 0)] = rho;
  c[tidx(1, 0, 0)] = R(0.5) * fh[0];
  c[tidx(0, 1, 0)] = R(0.5) * fh[1];
  c[tidx(0, 0, 1)] = R(0.5) * fh[2];
  c[tidx(2, 0, 0)] = R(0.5) * Q[0];
  c[tidx(0, 2, 0)] = R(0.5) * Q[1];
  c[tidx(0, 0, 2)] = R(0.5) * Q[2];
  c[tidx(1, 1, 0)] = R(0.25) * Q[3];
  c[tidx(1, 0, 1)] = R(0.25) * Q[4];
  c[tidx(0, 1, 1)] = R(0.25) * Q[5];
  c[tidx(0, 2, 2)] = R(1.0 / 12.0) * Q[0];
  c[tidx(2, 0, 2)] = R(1.0 / 12.0) * Q[1];
  c[tidx(2, 2, 0)] = R(1.0 / 12.0) * Q[2];
  c[tidx(1, 1, 2)] = R(-1.0 / 24.0) * Q[3];
  c[tidx(1, 2, 1)] = R(-1.0 / 24.0) * Q[4];
  c[tidx(2, 1, 1)] = R(-1.0 / 24.0) * Q[5];
  c[tidx(1, 2, 0)] = c[tidx(1, 0, 2)] = R(-1.0 / 12.0) * fh[0];
  c[tidx(2, 1, 0)] = c[tidx(0, 1, 2)] = R(-1.0 / 12.0) * fh[1];
  c[tidx(2, 0, 1)] = c[tidx(0, 2, 1)] = R(-1.0 / 12.0) * fh[2];
  c[tidx(1, 2, 2)] = R(1.0 / 72.0) * fh[0];
  c[tidx(2, 1, 2)] = R(1.0 / 72.0) * fh[1];
  c[tidx(2, 2, 1)] = R(1.0 / 72.0) * fh[2];
  c[tidx(1, 1, 1)] = c[tidx(2, 2, 2)] = R(0);
}

// Change of the Maxwell stress from the rest state, M(B) - M(b0), M = |B|^2/2 I - B B, as
// (xx, yy, zz, xy, xz, yz).
template <typename R>
FLAME_HD void maxwell_change(const R (&b)[3], const R (&b0)[3], R (&M)[6]) {
  const R dxx = b[0] * (R(2) * b0[0] + b[0]), dyy = b[1] * (R(2) * b0[1] + b[1]), dzz = b[2] * (R(2) * b0[2] + b[2]);
  M[0] = R(0.5) * (dyy + dzz - dxx);
  M[1] = R(0.5) * (dxx + dzz - dyy);
  M[2] = R(0.5) * (dxx + dyy - dzz);
  M[3] = -(b0[0] * b[1] + b[0] * (b0[1] + b[1]));
  M[4] = -(b0[0] * b[2] + b[0] * (b0[2] + b[2]));
  M[5] = -(b0[1] * b[2] + b[1] * (b0[2] + b[2]));
}

// Deviations of the populations from rest: coefficients about U (in a, consumed) plus the
// second-order part M, with drho in the place of the density coefficient.
template <typename R>
FLAME_HD void populate(R (&a)[kQ], R drho, const R (&U)[3], const R (&M)[6]) {
  shift_axis<0>(a, U[0]);
  shift_axis<1>(a, U[1]);
  shift_axis<2>(a, U[2]);
  a[tidx(0, 0, 0)] = drho;
  a[tidx(2, 0, 0)] += R(0.5) * M[0];
  a[tidx(0, 2, 0)] += R(0.5) * M[1];
  a[tidx(0, 0, 2)] += R(0.5) * M[2];
  a[tidx(1, 1, 0)] += R(0.25) * M[3];
  a[tidx(1, 0, 1)] += R(0.25) * M[4];
  a[tidx(0, 1, 1)] += R(0.25) * M[5];
  populate_axis<0>(a);
  populate_axis<1>(a);
  populate_axis<2>(a);
}

// Reverse of central_coefficients + maxwell_change + populate: l holds the adjoints of the 27
// populations in tensor order (consumed); returns those of the density (as d rho and in the
// coefficients alike), U, b and Q (up to a multiple of the identity, which tr Q = 0 takes out).
// The shift by u is exp(u N) with N lowering the order (N c)_1 = c_0, (N c)_2 = 2 c_1, so its
// derivative is N applied to the coefficients about U, of which only 25 are non-zero.
template <typename R>
FLAME_HD void populate_reverse(R (&l)[kQ], R rho, const R (&U)[3], const R (&Q)[6], const R (&fh)[3], const R (&B)[3],
                               R& lrho, R (&lU)[3], R (&lb)[3], R (&lQ)[6]) {
  populate_axis_t<2>(l);
  populate_axis_t<1>(l);
  populate_axis_t<0>(l);
  const R mxx = R(0.5) * l[tidx(2, 0, 0)], myy = R(0.5) * l[tidx(0, 2, 0)], mzz = R(0.5) * l[tidx(0, 0, 2)];
  const R mxy = R(0.25) * l[tidx(1, 1, 0)], mxz = R(0.25) * l[tidx(1, 0, 1)], myz = R(0.25) * l[tidx(0, 1, 1)];
  lb[0] = B[0] * (myy + mzz - mxx) - B[1] * mxy - B[2] * mxz;
  lb[1] = B[1] * (mxx + mzz - myy) - B[0] * mxy - B[2] * myz;
  lb[2] = B[2] * (mxx + myy - mzz) - B[0] * mxz - B[1] * myz;
  shift_axis_t<2>(l, U[2]);
  shift_axis_t<1>(l, U[1]);
  shift_axis_t<0>(l, U[0]);
  lrho = l[tidx(0, 0, 0)];
  lQ[0] = R(0.5) * l[tidx(2, 0, 0)] + R(1.0 / 12.0) * l[tidx(0, 2, 2)];
  lQ[1] = R(0.5) * l[tidx(0, 2, 0)] + R(1.0 / 12.0) * l[tidx(2, 0, 2)];
  lQ[2] = R(0.5) * l[tidx(0, 0, 2)] + R(1.0 / 12.0) * l[tidx(2, 2, 0)];
  lQ[3] = R(0.25) * l[tidx(1, 1, 0)] - R(1.0 / 24.0) * l[tidx(1, 1, 2)];
  lQ[4] = R(0.25) * l[tidx(1, 0, 1)] - R(1.0 / 24.0) * l[tidx(1, 2, 1)];
  lQ[5] = R(0.25) * l[tidx(0, 1, 1)] - R(1.0 / 24.0) * l[tidx(2, 1, 1)];
  R c[kQ];
  central_coefficients(rho, Q, fh, c);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int s = a == 0 ? 9 : a == 1 ? 3 : 1;
    R up = R(0), dn = R(0);
#pragma unroll
    for (int m = 0; m < 9; ++m) {
      const int i = a == 0 ? line_base<0>(m) : a == 1 ? line_base<1>(m) : line_base<2>(m);
      up += l[i + s] * c[i];
      if (i + s != tidx(1, 1, 1)) dn += l[i + 2 * s] * c[i + s];
    }
    lU[a] = R(0.5) * up + R(2) * dn;
  }
}

// Post-collision fluid deviations, in place (Sec. 3.1.2 with S = diag[1,1,1,1,w x5,1 x18]).
// Because every moment except the five deviatoric second-order ones relaxes to equilibrium
// with rate 1, the back-transform of the collided central moments is
//   f*_i = f^mhd(0)_i + (1 - w) sum_ab P_ab H^ab_i + sum_a (F_a/2) H^a_i,
// with P the deviatoric second central moment of f - f^mhd(0), H^ab = h..(c_x) h..(c_y) h..(c_z)
// the distributions with a single unit central moment, and F the body force (its half enters
// the velocity, the collision sets the first central moment to +F/2).
// In deviations: f^mhd(0)_i - f_rest_i = w_i [d rho E_i + (E_i - 1)] + (w_i / 2 c_s^4)
// (M(B) - M(b0)) : (c c - c_s^2 I), E_i = prod_a (1 + e_a), M(B) = |B|^2/2 I - B B.
//
// The tensor-product transforms above form the 27 directions: against one polynomial evaluation per
// direction they take the step from 1073 to 707 vector instructions and 265 to 172 registers (FP64, odd in place),
// the FP16 step at 384^3 from 5.55 to 5.04 ms and FP64 at 512^3 from 37.1 to 35.8 ms for an even
// and an odd step, and their FP32 error against FP64 is 30% smaller. (The second template argument has
// no effect.)
template <typename R, bool = true>
FLAME_HD void collide_fluid(R (&f)[kQ], const FluidMoments<R>& m, R rho,
                                              const R (&U)[3], const R (&b)[3], const R (&b0)[3],
                                              const R (&F)[3], R omega) {
  // deviatoric K = S2 - rho U U + (U F + F U)/2 + (B B - b0 b0); B B - b0 b0 = b0 b + b b0 + b b
  const R kxx = m.sxx - rho * U[0] * U[0] + U[0] * F[0] + b[0] * (R(2) * b0[0] + b[0]);
  const R kyy = m.syy - rho * U[1] * U[1] + U[1] * F[1] + b[1] * (R(2) * b0[1] + b[1]);
  const R kzz = m.szz - rho * U[2] * U[2] + U[2] * F[2] + b[2] * (R(2) * b0[2] + b[2]);
  const R om1 = R(1) - omega;
  const R tr = (kxx + kyy + kzz) * R(1.0 / 3.0);
  const R qxx = om1 * (kxx - tr), qyy = om1 * (kyy - tr), qzz = om1 * (kzz - tr);
  const R qxy = om1 * (m.sxy - rho * U[0] * U[1] + R(0.5) * (U[0] * F[1] + F[0] * U[1])
                       + b0[0] * b[1] + b[0] * b0[1] + b[0] * b[1]);
  const R qxz = om1 * (m.sxz - rho * U[0] * U[2] + R(0.5) * (U[0] * F[2] + F[0] * U[2])
                       + b0[0] * b[2] + b[0] * b0[2] + b[0] * b[2]);
  const R qyz = om1 * (m.syz - rho * U[1] * U[2] + R(0.5) * (U[1] * F[2] + F[1] * U[2])
                       + b0[1] * b[2] + b[1] * b0[2] + b[1] * b[2]);
  const R fhx = R(0.5) * F[0], fhy = R(0.5) * F[1], fhz = R(0.5) * F[2];
  R a[kQ], M[6];
  central_coefficients(rho, {qxx, qyy, qzz, qxy, qxz, qyz}, {fhx, fhy, fhz}, a);
  maxwell_change(b, b0, M);
  populate(a, m.drho, U, M);
#pragma unroll
  for (int i = 0; i < kQ; ++i) f[i] = a[tidx(cq(i, 0) + 1, cq(i, 1) + 1, cq(i, 2) + 1)];
}

// Post-collision magnetic deviations, in place (eq. MHD_LBscheme with the Hall equilibrium
// gHall_eq): g* = g - w_B (g - g^Hall(0)) + (1 - w_B/2) W_i S. With V = U - alpha J and
// E_ac = V_a B_c - B_a V_c, g^Hall(0)_{+-a, c} = W (B_c +- 4 E_ac), g^Hall(0)_{0, c} = W_0 B_c.
template <typename R>
FLAME_HD void collide_magnetic(R (&g)[kM], const R (&U)[3], const R (&B)[3],
                                                 const R (&b)[3], const R (&J)[3],
                                                 const R (&S)[3], R alpha, R omega_b) {
  const R V[3] = {U[0] - alpha * J[0], U[1] - alpha * J[1], U[2] - alpha * J[2]};
  const R src = R(1) - R(0.5) * omega_b;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const R eq0 = R(0.25) * b[c];
    g[c] = g[c] - omega_b * (g[c] - eq0) + src * R(0.25) * S[c];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const R E = (a == c) ? R(0) : (V[a] * B[c] - B[a] * V[c]);
      const R eqp = R(0.125) * (b[c] + R(4) * E);
      const R eqm = R(0.125) * (b[c] - R(4) * E);
      const int ip = (4 + a) * 3 + c, im = (1 + a) * 3 + c;
      g[ip] = g[ip] - omega_b * (g[ip] - eqp) + src * R(0.125) * S[c];
      g[im] = g[im] - omega_b * (g[im] - eqm) + src * R(0.125) * S[c];
    }
  }
}

// BGK variant of the fluid collision, in place on deviations: the central-moment step with every
// rate equal to w (Sec. 3.1.2; the standard operator of Sec. 3.1.1),
//   f*_i = f^mhd(0)_i + (1 - w)(f_i - f^mhd(0)_i) + (1 - w/2) sum_a F_a H^a_i.
// The force term ends the first central moments at +F/2 as in collide_fluid: before the
// collision those of f - f^mhd(0) are -F/2 (U carries F/2), and (1 - w) of them survive.
// f^mhd(0) - f_rest is the same equilibrium deviation as in collide_fluid.
template <typename R>
FLAME_HD void collide_fluid_bgk(R (&f)[kQ], const FluidMoments<R>& m, const R (&U)[3], const R (&b)[3],
                                const R (&b0)[3], const R (&F)[3], R omega) {
  // With T = f^mhd(0) + (1/w - 1/2) sum_a F_a H^a this is f* = T + (1 - w)(f - T), which keeps a
  // small f - T exact. Below w = 1 the force in T outgrows f, so there the form is f* = w T + (1 - w) f
  // (both terms positive weights of f), with the factor w taken into the coefficients.
  const bool slow = omega < R(1);
  const R om1 = R(1) - omega, s = slow ? omega : R(1), keep = slow ? R(0) : R(1);
  const R fk = (R(1) - R(0.5) * omega) / (slow ? R(1) : omega);   // w may be 0 in FP32
  R a[kQ], M[6];
  central_coefficients(s * (R(1) + m.drho), {R(0), R(0), R(0), R(0), R(0), R(0)}, {fk * F[0], fk * F[1], fk * F[2]}, a);
  maxwell_change(b, b0, M);
#pragma unroll
  for (int k = 0; k < 6; ++k) M[k] *= s;
  populate(a, s * m.drho, U, M);
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    const R t = a[tidx(cq(i, 0) + 1, cq(i, 1) + 1, cq(i, 2) + 1)];
    f[i] = t + om1 * (f[i] - keep * t);
  }
}

// ------------------------------------------------------------------ per-node reverse pass
// Vector-Jacobian product of one node's collision (the adjoint of collide_fluid +
// collide_magnetic with the moments and, on the moment route, J recomputed from the node's
// pre-collision deviations f, g). Given mf, mg = d loss / d(post-collision deviations), returns
// lf, lg = d loss / d(pre-collision deviations) through this node's collision, and lJ =
// d loss / dJ (stencil route: J is an input computed from neighbouring fields, Jst; on the moment
// route lJ is folded into lf, lg and returned as zero). F, S: forcing at the node.
// Forward quantities of one node that the reverse pass needs (recomputed from the pre-collision
// state; J from the moments on the moment route, else the J the forward step used).
template <typename R>
struct VjpState {
  FluidMoments<R> m;
  R rho, inv_rho, U[3], b[3], B[3], J[3], V[3], lam[3][3];
};

template <typename R, bool MOMENT>
FLAME_HD VjpState<R> vjp_forward(const R (&f)[kQ], const R (&g)[kM], const R (&F)[3], const R (&S)[3],
                                 const R (&Jst)[3], const PhysConst<R>& k) {
  VjpState<R> st;
  st.m = fluid_moments(f);
  st.rho = R(1) + st.m.drho;
  st.inv_rho = R(1) / st.rho;
  st.U[0] = (st.m.jx + R(0.5) * F[0]) * st.inv_rho;
  st.U[1] = (st.m.jy + R(0.5) * F[1]) * st.inv_rho;
  st.U[2] = (st.m.jz + R(0.5) * F[2]) * st.inv_rho;
  magnetic_moments(g, st.b, st.lam);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    st.b[c] += R(0.5) * S[c];
    st.B[c] = k.b0[c] + st.b[c];
  }
  if (MOMENT) current_from_moments(st.lam, st.U, st.B, k.alpha, k.omega_b, st.J);
  else { st.J[0] = Jst[0]; st.J[1] = Jst[1]; st.J[2] = Jst[2]; }
#pragma unroll
  for (int c = 0; c < 3; ++c) st.V[c] = st.U[c] - k.alpha * st.J[c];
  return st;
}

// Adjoints of a node's collision inputs, gathered from its outputs.
template <typename R>
struct NodeAdjoint {
  R lrho, lU[3], lb[3], ls2[6];
};

// Fluid half of the reverse pass: l, the adjoints of the 27 post-collision populations in tensor
// order, consumed. f* depends on rho, U, b and the second moments.
template <typename R>
FLAME_HD void vjp_fluid(const VjpState<R>& st, const R (&F)[3], const PhysConst<R>& k, R (&l)[kQ], NodeAdjoint<R>& o) {
  const FluidMoments<R>& m = st.m;
  const R rho = st.rho;
  const R(&U)[3] = st.U;
  const R(&b)[3] = st.b;
  const R(&B)[3] = st.B;
  const R(&b0)[3] = k.b0;
  const R om1 = R(1) - k.omega;
  const R kxx = m.sxx - rho * U[0] * U[0] + U[0] * F[0] + b[0] * (R(2) * b0[0] + b[0]);
  const R kyy = m.syy - rho * U[1] * U[1] + U[1] * F[1] + b[1] * (R(2) * b0[1] + b[1]);
  const R kzz = m.szz - rho * U[2] * U[2] + U[2] * F[2] + b[2] * (R(2) * b0[2] + b[2]);
  const R tr = (kxx + kyy + kzz) * R(1.0 / 3.0);
  const R Q[6] = {om1 * (kxx - tr), om1 * (kyy - tr), om1 * (kzz - tr),
                  om1 * (m.sxy - rho * U[0] * U[1] + R(0.5) * (U[0] * F[1] + F[0] * U[1])
                         + b0[0] * b[1] + b[0] * b0[1] + b[0] * b[1]),
                  om1 * (m.sxz - rho * U[0] * U[2] + R(0.5) * (U[0] * F[2] + F[0] * U[2])
                         + b0[0] * b[2] + b[0] * b0[2] + b[0] * b[2]),
                  om1 * (m.syz - rho * U[1] * U[2] + R(0.5) * (U[1] * F[2] + F[1] * U[2])
                         + b0[1] * b[2] + b[1] * b0[2] + b[1] * b[2])};
  R lQ[6];
  populate_reverse(l, rho, U, Q, {R(0.5) * F[0], R(0.5) * F[1], R(0.5) * F[2]}, B, o.lrho, o.lU, o.lb, lQ);
  // Q = (1 - w) (K - tr K / 3 I): the deviatoric projection is self-adjoint
  const R ltr = (lQ[0] + lQ[1] + lQ[2]) * R(1.0 / 3.0);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const R lk = om1 * (lQ[a] - ltr);
    o.ls2[a] = lk;
    o.lrho -= lk * U[a] * U[a];
    o.lU[a] += lk * (R(-2) * rho * U[a] + F[a]);
    o.lb[a] += lk * R(2) * B[a];
  }
  const int pa[3] = {0, 0, 1}, pb[3] = {1, 2, 2};
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const int a = pa[p], c = pb[p];
    const R lk = om1 * lQ[3 + p];
    o.ls2[3 + p] = lk;
    o.lrho -= lk * U[a] * U[c];
    o.lU[a] += lk * (-rho * U[c] + R(0.5) * F[c]);
    o.lU[c] += lk * (-rho * U[a] + R(0.5) * F[a]);
    o.lb[a] += lk * B[c];
    o.lb[c] += lk * B[a];
  }
}

// Magnetic half: mg, the adjoints of the post-collision magnetic populations, become those of the
// pre-collision ones; adds what reaches rho and U to o, and returns lJ (zero on the moment route,
// where J depends on the node's own moments).
template <typename R, bool MOMENT>
FLAME_HD void vjp_magnetic(const VjpState<R>& st, const PhysConst<R>& k, NodeAdjoint<R>& o, R (&mg)[kM], R (&lJ)[3]) {
  const R(&U)[3] = st.U;
  const R(&B)[3] = st.B;
  const R(&J)[3] = st.J;
  const R(&V)[3] = st.V;
  const R(&lam)[3][3] = st.lam;
  R(&lU)[3] = o.lU;
  R lb[3] = {o.lb[0], o.lb[1], o.lb[2]}, lB[3] = {R(0), R(0), R(0)};
  R lj0[3] = {R(0), R(0), R(0)};   // adjoint of eps:Lambda
  const R ob = k.omega_b;
  // g* = (1 - w_B) g + w_B g^Hall(0)(b, E) + source
  R lV[3] = {R(0), R(0), R(0)};
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    R acc = R(0.25) * ob * mg[c];
#pragma unroll
    for (int a = 0; a < 3; ++a) acc += R(0.125) * ob * (mg[(4 + a) * 3 + c] + mg[(1 + a) * 3 + c]);
    lb[c] += acc;
  }
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (a == c) continue;
      // g^Hall(0)_{+-a, c} = W (b_c +- 4 E_ac), W = 1/8, E_ac = V_a B_c - B_a V_c
      const R lE = R(0.5) * ob * (mg[(4 + a) * 3 + c] - mg[(1 + a) * 3 + c]);
      lV[a] += lE * B[c];
      lB[c] += lE * V[a];
      lB[a] -= lE * V[c];
      lV[c] -= lE * B[a];
    }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    lU[a] += lV[a];
    lJ[a] = -k.alpha * lV[a];
  }
  // current from the moments: J = N / D, N = r - kk r x B + kk^2 (r.B) B, D = 1 + kk^2 |B|^2,
  // r = -4 w_B J0, J0 = A(Lambda) - 2 U x B
  if (MOMENT) {
    const R kk = R(8) * k.alpha * k.omega_b;
    const R kk2 = kk * kk;
    const R D = R(1) + kk2 * (B[0] * B[0] + B[1] * B[1] + B[2] * B[2]);
    const R j0[3] = {lam[1][2] - lam[2][1] - R(2) * (U[1] * B[2] - U[2] * B[1]),
                     lam[2][0] - lam[0][2] - R(2) * (U[2] * B[0] - U[0] * B[2]),
                     lam[0][1] - lam[1][0] - R(2) * (U[0] * B[1] - U[1] * B[0])};
    const R r[3] = {R(-4) * k.omega_b * j0[0], R(-4) * k.omega_b * j0[1], R(-4) * k.omega_b * j0[2]};
    const R inv = R(1) / D;
    const R lN[3] = {lJ[0] * inv, lJ[1] * inv, lJ[2] * inv};
    const R lD = -(lJ[0] * J[0] + lJ[1] * J[1] + lJ[2] * J[2]) * inv;
    const R BlN = B[0] * lN[0] + B[1] * lN[1] + B[2] * lN[2];
    const R rB = r[0] * B[0] + r[1] * B[1] + r[2] * B[2];
    // d/dr:  lN - kk (B x lN) + kk^2 (B.lN) B
    const R Bxl[3] = {B[1] * lN[2] - B[2] * lN[1], B[2] * lN[0] - B[0] * lN[2], B[0] * lN[1] - B[1] * lN[0]};
    R lr[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) lr[a] = lN[a] - kk * Bxl[a] + kk2 * BlN * B[a];
    // d/dB: -kk (lN x r) + kk^2 ((B.lN) r + (r.B) lN) + 2 kk^2 lD B
    const R lxr[3] = {lN[1] * r[2] - lN[2] * r[1], lN[2] * r[0] - lN[0] * r[2], lN[0] * r[1] - lN[1] * r[0]};
#pragma unroll
    for (int a = 0; a < 3; ++a) lB[a] += -kk * lxr[a] + kk2 * (BlN * r[a] + rB * lN[a]) + R(2) * kk2 * lD * B[a];
#pragma unroll
    for (int a = 0; a < 3; ++a) lj0[a] = R(-4) * k.omega_b * lr[a];
    // J0 = A - 2 U x B: d/dU = -2 (B x lj0), d/dB = -2 (lj0 x U)
    const R Bxj[3] = {B[1] * lj0[2] - B[2] * lj0[1], B[2] * lj0[0] - B[0] * lj0[2], B[0] * lj0[1] - B[1] * lj0[0]};
    const R jxU[3] = {lj0[1] * U[2] - lj0[2] * U[1], lj0[2] * U[0] - lj0[0] * U[2], lj0[0] * U[1] - lj0[1] * U[0]};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      lU[a] += R(-2) * Bxj[a];
      lB[a] += R(-2) * jxU[a];
    }
    lJ[0] = lJ[1] = lJ[2] = R(0);
  }
  // b_c = sum_i g_ic (+ S/2), Lambda_ac = g_{+a,c} - g_{-a,c}, (eps:Lambda)_e = Lambda_ac - Lambda_ca
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    lb[c] += lB[c];
    mg[c] = (R(1) - ob) * mg[c] + lb[c];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      R& p = mg[(4 + a) * 3 + c];
      R& q = mg[(1 + a) * 3 + c];
      p = (R(1) - ob) * p + lb[c];
      q = (R(1) - ob) * q + lb[c];
      if (MOMENT && a != c) {
        const int e = 3 - a - c;
        const R l = (a + 1) % 3 == c ? lj0[e] : -lj0[e];
        p += l;
        q -= l;
      }
    }
  }
}

// Adjoints of the pre-collision fluid populations: U = (j + F/2) / rho, d rho = sum f,
// j = sum f c, S2 = sum f c c; formed axis by axis.
template <typename R>
FLAME_HD void vjp_fluid_populations(const VjpState<R>& st, const NodeAdjoint<R>& o, R (&lf)[kQ]) {
  const R lj[3] = {o.lU[0] * st.inv_rho, o.lU[1] * st.inv_rho, o.lU[2] * st.inv_rho};
  const R l0 = o.lrho - (o.lU[0] * st.U[0] + o.lU[1] * st.U[1] + o.lU[2] * st.U[2]) * st.inv_rho;
  auto at = [](R c0, R c1, R c2, int x) { return x == 0 ? c0 : x > 0 ? c0 + (c2 + c1) : c0 + (c2 - c1); };
  auto lin = [](R c0, R c1, int x) { return x == 0 ? c0 : x > 0 ? c0 + c1 : c0 - c1; };
#pragma unroll
  for (int x = -1; x <= 1; ++x) {
    const R px = at(l0, lj[0], o.ls2[0], x), qy = lin(lj[1], o.ls2[3], x), qz = lin(lj[2], o.ls2[4], x);
#pragma unroll
    for (int y = -1; y <= 1; ++y) {
      const R pxy = at(px, qy, o.ls2[1], y), rz = lin(qz, o.ls2[5], y);
#pragma unroll
      for (int z = -1; z <= 1; ++z) lf[qindex(x, y, z)] = at(pxy, rz, o.ls2[2], z);
    }
  }
}

template <typename R, bool MOMENT>
FLAME_HD void collide_vjp(const R (&f)[kQ], const R (&g)[kM], const R (&F)[3], const R (&S)[3],
                          const R (&Jst)[3], const PhysConst<R>& k, const R (&mf)[kQ], const R (&mg)[kM],
                          R (&lf)[kQ], R (&lg)[kM], R (&lJ)[3]) {
  const VjpState<R> st = vjp_forward<R, MOMENT>(f, g, F, S, Jst, k);
  R l[kQ];
#pragma unroll
  for (int i = 0; i < kQ; ++i) l[tidx(cq(i, 0) + 1, cq(i, 1) + 1, cq(i, 2) + 1)] = mf[i];
  NodeAdjoint<R> o;
  vjp_fluid(st, F, k, l, o);
#pragma unroll
  for (int q = 0; q < kM; ++q) lg[q] = mg[q];
  vjp_magnetic<R, MOMENT>(st, k, o, lg, lJ);
  vjp_fluid_populations(st, o, lf);
}

// ------------------------------------------------------------------ initial state of a node
// Deviations of the initial populations at a node (rho = 1): fluid f^mhd(0)(1, u, B) plus the
// first-order non-equilibrium stress P0 = -(c_s^2 / w)(G + G^T - 2/3 tr G I), G = grad u, and
// -F/2 first central moment; magnetic g^Hall(0)(u, B, curl b) - (1/w_B) W_i xi_ia d_a b_c - S/2 W_i
// (with u taken as zero in g^Hall(0) for electron MHD).
// G[a][c] = d u_c / d x_a, H[a][c] = d b_c / d x_a (ignored unless the flags say present).
struct InitFlags {
  bool fluid_noneq;   // add the fluid non-equilibrium stress (needs G)
  bool mag_noneq;     // add the magnetic non-equilibrium part (needs H)
  bool has_H;         // J = curl b from H (else J = 0)
  bool emhd = false;  // electron MHD: the magnetic equilibrium without the bulk velocity
};

FLAME_HD void init_node(const double (&u)[3], const double (&b)[3], const double (&G)[3][3],
                        const double (&H)[3][3], const double (&F)[3], const double (&S)[3],
                        const PhysConst<double>& k, InitFlags fl, double (&f)[kQ], double (&g)[kM]) {
  const double B[3] = {k.b0[0] + b[0], k.b0[1] + b[1], k.b0[2] + b[2]};
  double P[3][3] = {};
  if (fl.fluid_noneq) {
    const double div = G[0][0] + G[1][1] + G[2][2];
    const double s = -(1.0 / 3.0) / k.omega;
    for (int p = 0; p < 3; ++p)
      for (int q = 0; q < 3; ++q) P[p][q] = s * (G[p][q] + G[q][p] - (p == q ? 2.0 / 3.0 * div : 0.0));
  }
  const Axis<double> ax(u[0]), ay(u[1]), az(u[2]);
  const double sb = k.b0[0] * b[0] + k.b0[1] * b[1] + k.b0[2] * b[2] + 0.5 * (b[0] * b[0] + b[1] * b[1] + b[2] * b[2]);
  for (int i = 0; i < kQ; ++i) {
    const int x = cq(i, 0) + 1, y = cq(i, 1) + 1, z = cq(i, 2) + 1;
    const double ex = ax.e[x], ey = ay.e[y], ez = az.e[z];
    const double em1 = ex + (1.0 + ex) * (ey + (1.0 + ey) * ez);
    const double w = wq(i);
    double v = w * em1;
    const double bc = cq(i, 0) * b[0] + cq(i, 1) * b[1] + cq(i, 2) * b[2];
    const double b0c = cq(i, 0) * k.b0[0] + cq(i, 1) * k.b0[1] + cq(i, 2) * k.b0[2];
    v += w * 4.5 * (sb * (speed2q(i) - 1.0 / 3.0) - bc * (2.0 * b0c + bc));
    const double h0x = ax.h0[x], h0y = ay.h0[y], h0z = az.h0[z];
    const double h1x = ax.h1[x], h1y = ay.h1[y], h1z = az.h1[z];
    const double h2x = ax.h2[x], h2y = ay.h2[y], h2z = az.h2[z];
    v += P[0][0] * h2x * h0y * h0z + P[1][1] * h0x * h2y * h0z + P[2][2] * h0x * h0y * h2z
       + P[0][1] * h1x * h1y * h0z + P[0][2] * h1x * h0y * h1z + P[1][2] * h0x * h1y * h1z;
    v -= 0.5 * (F[0] * h1x * h0y * h0z + F[1] * h0x * h1y * h0z + F[2] * h0x * h0y * h1z);
    f[i] = v;
  }
  double J[3] = {0, 0, 0};
  if (fl.has_H) {
    J[0] = H[1][2] - H[2][1];
    J[1] = H[2][0] - H[0][2];
    J[2] = H[0][1] - H[1][0];
  }
  const double um = fl.emhd ? 0.0 : 1.0;
  const double V[3] = {um * u[0] - k.alpha * J[0], um * u[1] - k.alpha * J[1], um * u[2] - k.alpha * J[2]};
  for (int i = 0; i < 7; ++i)
    for (int c = 0; c < 3; ++c) {
      double xv = 0, xb = 0, xg = 0;
      for (int p = 0; p < 3; ++p) {
        xv += xim(i, p) * V[p];
        xb += xim(i, p) * B[p];
        xg += xim(i, p) * H[p][c];
      }
      double v = wm(i) * (b[c] + 4.0 * (xv * B[c] - xb * V[c]));
      if (fl.mag_noneq) v -= wm(i) * xg / k.omega_b;
      v -= 0.5 * wm(i) * S[c];
      g[i * 3 + c] = v;
    }
}

// Vector-Jacobian product of init_node: lf, lg = d loss / d(initial deviations) ->
// gu, gb, gG, gH = d loss / d(u, b, G, H) at the node.
FLAME_HD void init_node_vjp(const double (&u)[3], const double (&b)[3], const double (&G)[3][3],
                            const double (&H)[3][3], const double (&F)[3], const PhysConst<double>& k,
                            InitFlags fl, const double (&lf)[kQ], const double (&lg)[kM], double (&gu)[3],
                            double (&gb)[3], double (&gG)[3][3], double (&gH)[3][3]) {
  const double B[3] = {k.b0[0] + b[0], k.b0[1] + b[1], k.b0[2] + b[2]};
  for (int a = 0; a < 3; ++a) {
    gu[a] = gb[a] = 0.0;
    for (int c = 0; c < 3; ++c) gG[a][c] = gH[a][c] = 0.0;
  }
  double P[3][3] = {};
  const double s = -(1.0 / 3.0) / k.omega;
  if (fl.fluid_noneq) {
    const double div = G[0][0] + G[1][1] + G[2][2];
    for (int p = 0; p < 3; ++p)
      for (int q = 0; q < 3; ++q) P[p][q] = s * (G[p][q] + G[q][p] - (p == q ? 2.0 / 3.0 * div : 0.0));
  }
  double l[kQ], lrho, lP[6];   // xx, yy, zz, xy, xz, yz
#pragma unroll
  for (int i = 0; i < kQ; ++i) l[tidx(cq(i, 0) + 1, cq(i, 1) + 1, cq(i, 2) + 1)] = lf[i];
  populate_reverse(l, 1.0, u, {P[0][0], P[1][1], P[2][2], P[0][1], P[0][2], P[1][2]},
                   {-0.5 * F[0], -0.5 * F[1], -0.5 * F[2]}, B, lrho, gu, gb, lP);
  if (fl.fluid_noneq) {
    const double ltr = lP[0] + lP[1] + lP[2];
    for (int a = 0; a < 3; ++a) gG[a][a] += s * (2.0 * lP[a] - 2.0 / 3.0 * ltr);
    gG[0][1] += s * lP[3]; gG[1][0] += s * lP[3];
    gG[0][2] += s * lP[4]; gG[2][0] += s * lP[4];
    gG[1][2] += s * lP[5]; gG[2][1] += s * lP[5];
  }
  double J[3] = {0, 0, 0};
  if (fl.has_H) {
    J[0] = H[1][2] - H[2][1];
    J[1] = H[2][0] - H[0][2];
    J[2] = H[0][1] - H[1][0];
  }
  const double V[3] = {u[0] - k.alpha * J[0], u[1] - k.alpha * J[1], u[2] - k.alpha * J[2]};
  double lV[3] = {0, 0, 0};
  for (int i = 0; i < 7; ++i)
    for (int c = 0; c < 3; ++c) {
      const double mu = lg[i * 3 + c];
      const double W = wm(i);
      double xv = 0, xb = 0;
      for (int p = 0; p < 3; ++p) {
        xv += xim(i, p) * V[p];
        xb += xim(i, p) * B[p];
      }
      gb[c] += mu * W * (1.0 + 4.0 * xv);
      lV[c] -= mu * 4.0 * W * xb;
      for (int d = 0; d < 3; ++d) {
        gb[d] -= mu * 4.0 * W * xim(i, d) * V[c];
        lV[d] += mu * 4.0 * W * xim(i, d) * B[c];
        if (fl.mag_noneq) gH[d][c] -= mu * W * xim(i, d) / k.omega_b;
      }
    }
  for (int a = 0; a < 3; ++a) gu[a] += lV[a];
  if (fl.has_H) {
    const double lJ[3] = {-k.alpha * lV[0], -k.alpha * lV[1], -k.alpha * lV[2]};
    gH[1][2] += lJ[0]; gH[2][1] -= lJ[0];
    gH[2][0] += lJ[1]; gH[0][2] -= lJ[1];
    gH[0][1] += lJ[2]; gH[1][0] -= lJ[2];
  }
}

// Periodic neighbour of a node.
FLAME_HD int wrap(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

}  // namespace flame
