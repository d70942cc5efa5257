// C ABI of the library (include/flame.h): validation, buffer bookkeeping, the initial
// state, canonical access, node fields, FP64 reductions and shell spectra.

#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "flame_access.h"
#include "flame_internal.h"

namespace flame {

// Rest populations f^mhd(0)(1, 0, b0), passed to kernels by value.
struct Rest {
  double f[27];
  double b0[3];
};

// ------------------------------------------------------------------ canonical view
// Read access to the current state in canonical order, for the auxiliary kernels. Returns
// decoded deviations as double.
template <typename S>
struct View {
  const S* F;
  const S* G;
  // addressing of the canonical population i at node x:
  //   0: slot i at x (AA even step); 1: slot opp(i) at x - c_i (AA odd step);
  //   2: slot i at x - c_i (two-lattice pull: the source copy holds post-collision values)
  int fmode;
  int gmode;
  int nx, ny, nz;
  size_t n;
  size_t stride;   // elements between population arrays

  // node index in 32-bit arithmetic: flame_init refuses grids of 2^32 nodes or more
  __device__ size_t node(int x, int y, int z) const {
    return (static_cast<size_t>(z) * ny + y) * nx + x;
  }
  // canonical population i (component c) of node (x, y, z), with the addressing mode fixed at compile
  // time (no branch per access, so that a
  // node's loads can all be in flight together)
  template <int M>
  __device__ double fm(int i, int x, int y, int z) const {
    const size_t idx = M == 0 ? static_cast<size_t>(i) * stride + node(x, y, z)
                              : static_cast<size_t>(M == 1 ? oppq(i) : i) * stride +
                                    node(wrap(x - cq(i, 0), nx), wrap(y - cq(i, 1), ny), wrap(z - cq(i, 2), nz));
    return static_cast<double>(F[idx]) / Enc<S>::fscale(i);
  }
  template <int M>
  __device__ double gm(int i, int c, int x, int y, int z) const {
    const size_t idx = M == 0 ? static_cast<size_t>(i * 3 + c) * stride + node(x, y, z)
                              : static_cast<size_t>((M == 1 ? oppm(i) : i) * 3 + c) * stride +
                                    node(wrap(x - xim(i, 0), nx), wrap(y - xim(i, 1), ny), wrap(z - xim(i, 2), nz));
    return static_cast<double>(G[idx]) / Enc<S>::mscale(i);
  }
  // runtime mode: the element index is selected, then one load
  __device__ double f(int i, int x, int y, int z) const {
    size_t idx = fmode == 0 ? static_cast<size_t>(i) * stride + node(x, y, z)
                            : static_cast<size_t>(fmode == 1 ? oppq(i) : i) * stride +
                                  node(wrap(x - cq(i, 0), nx), wrap(y - cq(i, 1), ny), wrap(z - cq(i, 2), nz));
    return static_cast<double>(F[idx]) / Enc<S>::fscale(i);
  }
  __device__ double g(int i, int c, int x, int y, int z) const {
    size_t idx = gmode == 0 ? static_cast<size_t>(i * 3 + c) * stride + node(x, y, z)
                            : static_cast<size_t>((gmode == 1 ? oppm(i) : i) * 3 + c) * stride +
                                  node(wrap(x - xim(i, 0), nx), wrap(y - xim(i, 1), ny), wrap(z - xim(i, 2), nz));
    return static_cast<double>(G[idx]) / Enc<S>::mscale(i);
  }
};

// All populations of node (x, y, z), decoded, in canonical order; the mode switch is taken once
// per node.
template <int M, typename S>
__device__ __forceinline__ void view_fluid(const View<S>& v, int x, int y, int z, double (&f)[kQ]) {
#pragma unroll
  for (int i = 0; i < kQ; ++i) f[i] = v.template fm<M>(i, x, y, z);
}
template <int M, typename S>
__device__ __forceinline__ void view_magnetic(const View<S>& v, int x, int y, int z, double (&g)[kM]) {
#pragma unroll
  for (int i = 0; i < 7; ++i)
#pragma unroll
    for (int c = 0; c < 3; ++c) g[i * 3 + c] = v.template gm<M>(i, c, x, y, z);
}
template <typename S>
__device__ __forceinline__ void view_node(const View<S>& v, int x, int y, int z, double (&f)[kQ], double (&g)[kM]) {
  if (v.fmode == 0) view_fluid<0>(v, x, y, z, f);
  else if (v.fmode == 1) view_fluid<1>(v, x, y, z, f);
  else view_fluid<2>(v, x, y, z, f);
  if (v.gmode == 0) view_magnetic<0>(v, x, y, z, g);
  else if (v.gmode == 1) view_magnetic<1>(v, x, y, z, g);
  else view_magnetic<2>(v, x, y, z, g);
}

// Where a writer of the canonical state (initial state, set) puts population i of node
// (x, y, z): its own slot for in-place sets; for pull sets the slot at x - c_i, which is where
// the next step at node x pulls population i from.
struct Placement {
  bool fpull, gpull;
  int nx, ny, nz;
  __device__ size_t f(int i, int x, int y, int z) const {
    if (fpull) { x = wrap(x - cq(i, 0), nx); y = wrap(y - cq(i, 1), ny); z = wrap(z - cq(i, 2), nz); }
    return (static_cast<size_t>(z) * ny + y) * nx + x;
  }
  __device__ size_t g(int i, int x, int y, int z) const {
    if (gpull) { x = wrap(x - xim(i, 0), nx); y = wrap(y - xim(i, 1), ny); z = wrap(z - xim(i, 2), nz); }
    return (static_cast<size_t>(z) * ny + y) * nx + x;
  }
};

// Node quantities in FP64 from the canonical view.
struct NodeQ {
  double rho, U[3], B[3], b[3], J[3], divb;
  bool finite;
};

template <typename S>
struct AuxArgs {
  View<S> v;
  const typename Enc<S>::R* force_u;
  const typename Enc<S>::R* force_b;
  double b0[3];
  double alpha, omega_b;
  int emhd;     // electron MHD: J from the moments with the bulk velocity taken as zero
};

// Component comp of b, with the magnetic addressing mode fixed at compile time.
template <int M, typename S>
__device__ __forceinline__ double field_fluct_m(const AuxArgs<S>& a, int comp, int x, int y, int z) {
  double s = a.v.template gm<M>(0, comp, x, y, z);
#pragma unroll
  for (int i = 1; i < 7; ++i) s += a.v.template gm<M>(i, comp, x, y, z);
  if (a.force_b) s += 0.5 * static_cast<double>(a.force_b[static_cast<size_t>(comp) * a.v.n + a.v.node(x, y, z)]);
  return s;
}
// On the moment route (the curl-stencil route has stencil_march_kernel).
template <typename S>
__device__ NodeQ node_quantities(const AuxArgs<S>& a, int x, int y, int z) {
  NodeQ q;
  const View<S>& v = a.v;
  const size_t cell = v.node(x, y, z);
  // unrolled, so that f and g stay in registers (a runtime index would put them in per-thread private memory)
  double f[kQ], g[kM];
  view_node(v, x, y, z, f, g);
  bool fin = true;
#pragma unroll
  for (int i = 0; i < kQ; ++i) fin = fin && isfinite(f[i]);
#pragma unroll
  for (int k = 0; k < kM; ++k) fin = fin && isfinite(g[k]);
  q.finite = fin;
  double drho = 0, j[3] = {0, 0, 0};
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    drho += f[i];
#pragma unroll
    for (int c = 0; c < 3; ++c) j[c] += cq(i, c) * f[i];
  }
  q.rho = 1.0 + drho;
  for (int c = 0; c < 3; ++c) {
    const double F = a.force_u ? static_cast<double>(a.force_u[static_cast<size_t>(c) * v.n + cell]) : 0.0;
    q.U[c] = (j[c] + 0.5 * F) / q.rho;
  }
  double lam[3][3];
  double bb[3];
  magnetic_moments(g, bb, lam);
  for (int c = 0; c < 3; ++c) {
    const double src = a.force_b ? static_cast<double>(a.force_b[static_cast<size_t>(c) * v.n + cell]) : 0.0;
    q.b[c] = bb[c] + 0.5 * src;
    q.B[c] = a.b0[c] + q.b[c];
  }
  const double zero[3] = {0.0, 0.0, 0.0};
  current_from_moments(lam, a.emhd ? zero : q.U, q.B, a.alpha, a.omega_b, q.J);
  q.divb = -4.0 * a.omega_b * (lam[0][0] + lam[1][1] + lam[2][2]);
  return q;
}

// cell < 2^32 (flame_init refuses larger grids), so 32-bit division suffices
__device__ __forceinline__ void node_xyz(size_t cell, int nx, int ny, int& x, int& y, int& z) {
  x = static_cast<int>(cell % nx);
  const size_t r = cell / nx;
  y = static_cast<int>(r % ny);
  z = static_cast<int>(r / ny);
}

// ------------------------------------------------------------------ initial state
template <typename S>
struct InitArgs {
  using R = typename Enc<S>::R;
  S* F;
  S* G;
  const double* u;
  const double* b;
  const double* gu;   // [3][3][n] or null
  const double* gb;
  const R* force_u;
  const R* force_b;
  double b0[3];
  double omega, omega_b, alpha;
  int noneq;
  int emhd;
  int nx, ny, nz;
  size_t n;
  size_t stride;
  Placement at;
};

template <typename S>
__global__ __launch_bounds__(256) void init_kernel(InitArgs<S> a) {
  using E = Enc<S>;
  const size_t cell = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (cell >= a.n) return;
  const size_t n = a.n;
  int px, py, pz;
  node_xyz(cell, a.nx, a.ny, px, py, pz);
  double U[3], b[3], B[3], F[3] = {0, 0, 0}, Sb[3] = {0, 0, 0};
  for (int c = 0; c < 3; ++c) {
    U[c] = a.u[c * n + cell];
    b[c] = a.b[c * n + cell];
    B[c] = a.b0[c] + b[c];
    if (a.force_u) F[c] = static_cast<double>(a.force_u[c * n + cell]);
    if (a.force_b) Sb[c] = static_cast<double>(a.force_b[c * n + cell]);
  }
  // gradients: given, or (with the non-equilibrium initialisation) central differences on the grid
  auto central = [&](const double* v, double (&g)[3][3]) {
    auto at = [&](int x, int y, int z) { return (static_cast<size_t>(z) * a.ny + y) * a.nx + x; };
    const size_t xm = at(wrap(px - 1, a.nx), py, pz), xp = at(wrap(px + 1, a.nx), py, pz);
    const size_t ym = at(px, wrap(py - 1, a.ny), pz), yp = at(px, wrap(py + 1, a.ny), pz);
    const size_t zm = at(px, py, wrap(pz - 1, a.nz)), zp = at(px, py, wrap(pz + 1, a.nz));
    for (int c = 0; c < 3; ++c) {
      const double* vc = v + c * n;
      g[0][c] = 0.5 * (vc[xp] - vc[xm]);
      g[1][c] = 0.5 * (vc[yp] - vc[ym]);
      g[2][c] = 0.5 * (vc[zp] - vc[zm]);
    }
  };
  double gu[3][3] = {}, gb[3][3] = {};
  bool have_gu = a.gu != nullptr, have_gb = a.gb != nullptr;
  if (a.gu) {
    for (int p = 0; p < 3; ++p)
      for (int q = 0; q < 3; ++q) gu[p][q] = a.gu[(p * 3 + q) * n + cell];
  } else if (a.noneq) {
    central(a.u, gu);
    have_gu = true;
  }
  if (a.gb) {
    for (int p = 0; p < 3; ++p)
      for (int q = 0; q < 3; ++q) gb[p][q] = a.gb[(p * 3 + q) * n + cell];
  } else if (a.noneq) {
    central(a.b, gb);
    have_gb = true;
  }
  PhysConst<double> k;
  k.omega = a.omega;
  k.omega_b = a.omega_b;
  k.alpha = a.alpha;
  for (int c = 0; c < 3; ++c) k.b0[c] = a.b0[c];
  InitFlags fl;
  fl.fluid_noneq = a.noneq && have_gu;
  fl.mag_noneq = a.noneq && have_gb;
  fl.has_H = have_gb;
  fl.emhd = a.emhd != 0;
  double f[kQ], g[kM];
  init_node(U, b, gu, gb, F, Sb, k, fl, f, g);
  for (int i = 0; i < kQ; ++i)
    a.F[static_cast<size_t>(i) * a.stride + a.at.f(i, px, py, pz)] = E::enc(f[i], E::fscale(i));
  for (int i = 0; i < 7; ++i)
    for (int c = 0; c < 3; ++c)
      a.G[static_cast<size_t>(i * 3 + c) * a.stride + a.at.g(i, px, py, pz)] = E::enc(g[i * 3 + c], E::mscale(i));
}

// ------------------------------------------------------------------ canonical copies
template <typename S>
__global__ __launch_bounds__(256) void get_kernel(View<S> v, Rest r, double* dst) {
  const size_t cell = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (cell >= v.n) return;
  int x, y, z;
  node_xyz(cell, v.nx, v.ny, x, y, z);
  for (int i = 0; i < kQ; ++i) dst[static_cast<size_t>(i) * v.n + cell] = r.f[i] + v.f(i, x, y, z);
  for (int i = 0; i < 7; ++i)
    for (int c = 0; c < 3; ++c)
      dst[(27 + static_cast<size_t>(i * 3 + c)) * v.n + cell] = wm(i) * r.b0[c] + v.g(i, c, x, y, z);
}

template <typename S>
__global__ __launch_bounds__(256) void set_kernel(S* F, S* G, size_t n, size_t stride, Placement at, Rest r,
                                                  const double* src) {
  using E = Enc<S>;
  const size_t cell = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (cell >= n) return;
  int x, y, z;
  node_xyz(cell, at.nx, at.ny, x, y, z);
  for (int i = 0; i < kQ; ++i)
    F[static_cast<size_t>(i) * stride + at.f(i, x, y, z)] =
        E::enc(src[static_cast<size_t>(i) * n + cell] - r.f[i], E::fscale(i));
  for (int i = 0; i < 7; ++i)
    for (int c = 0; c < 3; ++c) {
      const size_t k = static_cast<size_t>(i * 3 + c);
      G[k * stride + at.g(i, x, y, z)] = E::enc(src[(27 + k) * n + cell] - wm(i) * r.b0[c], E::mscale(i));
    }
}

// Trace lattice of the current state (two-lattice pull layout, node stride n): slot i at x holds
// canonical population i of node x + c_i, which a pull step there reads. In place that is slot i at
// x + c_i after an even number of steps (M 0) and slot opp(i) at x after an odd one (M 1). The stored
// values are moved without decoding, so the copy is exact. Bound by HBM; written in whole lines (128^3 FP32
// 257 us when each node wrote to x - c_i through 64-bit indices, 204 now; 48^3 FP64 27 and 17).
template <typename S, int M>
__global__ __launch_bounds__(kRowThreadsMax) void export_kernel(const S* F, const S* G, size_t stride, GridShape shape,
                                                                size_t n, S* lat) {
  constexpr Addr A = Addr::Global;
  uint32_t cell;
  if (!own_cell(shape, cell)) return;
  const NodeAt at = NodeAt::of(cell, shape);
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    const uint32_t off = M == 0 ? at.rw.at(cq(i, 0), cq(i, 1)) + at.pl.at(cq(i, 2)) : cell;
    st<A>(lat + static_cast<size_t>(i) * n, cell, ld<A>(F + static_cast<size_t>(M == 0 ? i : oppq(i)) * stride, off));
  }
#pragma unroll
  for (int i = 0; i < 7; ++i) {
    const uint32_t off = M == 0 ? at.rw.at(xim(i, 0), xim(i, 1)) + at.pl.at(xim(i, 2)) : cell;
#pragma unroll
    for (int c = 0; c < 3; ++c)
      st<A>(lat + static_cast<size_t>(kQ + i * 3 + c) * n, cell,
            ld<A>(G + static_cast<size_t>((M == 0 ? i : oppm(i)) * 3 + c) * stride, off));
  }
}

template <typename S>
__global__ __launch_bounds__(256) void gather_kernel(View<S> v, Rest r, const int64_t* cells, int64_t cnt,
                                                     double* out) {
  const int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k >= cnt) return;
  const int64_t cell = cells[k];
  if (cell < 0 || static_cast<size_t>(cell) >= v.n) {
    for (int q = 0; q < 48; ++q) out[k * 48 + q] = NAN;
    return;
  }
  int x, y, z;
  node_xyz(static_cast<size_t>(cell), v.nx, v.ny, x, y, z);
  for (int i = 0; i < kQ; ++i) out[k * 48 + i] = r.f[i] + v.f(i, x, y, z);
  for (int i = 0; i < 7; ++i)
    for (int c = 0; c < 3; ++c) out[k * 48 + 27 + i * 3 + c] = wm(i) * r.b0[c] + v.g(i, c, x, y, z);
}

// ------------------------------------------------------------------ node fields
template <typename S>
__global__ __launch_bounds__(256) void moments_kernel(AuxArgs<S> a, double* rho, double* u, double* B,
                                                      double* J, double* divb) {
  const size_t cell = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (cell >= a.v.n) return;
  int x, y, z;
  node_xyz(cell, a.v.nx, a.v.ny, x, y, z);
  const NodeQ q = node_quantities(a, x, y, z);
  const size_t n = a.v.n;
  if (rho) rho[cell] = q.rho;
  if (divb) divb[cell] = q.divb;
  for (int c = 0; c < 3; ++c) {
    if (u) u[c * n + cell] = q.U[c];
    if (B) B[c * n + cell] = q.B[c];
    if (J) J[c * n + cell] = q.J[c];
  }
}

// ------------------------------------------------------------------ adjoint of the node fields
// lam = d loss / d(canonical deviations) for a loss of the node fields u = (j + F/2) / rho and
// B = b0 + sum g + S/2: du_a / df_i = (c_ia - u_a) / rho, dB_c / dg_{i,c} = 1.
template <typename S>
__global__ __launch_bounds__(256) void adjoint_fields_kernel(View<S> v, const typename Enc<S>::R* force_u,
                                                             const double* dl_du, const double* dl_db,
                                                             typename Enc<S>::R* lam) {
  using R = typename Enc<S>::R;
  const size_t cell = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (cell >= v.n) return;
  const size_t n = v.n;
  int x, y, z;
  node_xyz(cell, v.nx, v.ny, x, y, z);
  double lu[3] = {0, 0, 0}, U[3] = {0, 0, 0}, rho = 1.0;
  if (dl_du) {
    double f[kQ], j[3] = {0, 0, 0};
    if (v.fmode == 0) view_fluid<0>(v, x, y, z, f);
    else if (v.fmode == 1) view_fluid<1>(v, x, y, z, f);
    else view_fluid<2>(v, x, y, z, f);
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
      rho += f[i];
#pragma unroll
      for (int c = 0; c < 3; ++c) j[c] += cq(i, c) * f[i];   // also where c is 0: an infinity makes U NaN
    }
    for (int c = 0; c < 3; ++c) {
      const double F = force_u ? static_cast<double>(force_u[c * n + cell]) : 0.0;
      U[c] = (j[c] + 0.5 * F) / rho;
      lu[c] = dl_du[c * n + cell];
    }
  }
  // unrolled, so that the node's loads are in flight together and its velocities are constants (48^3 FP64
  // 30 us with loops over a table of velocities, 16 now)
  const double inv_rho = 1.0 / rho;
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) s += lu[c] * (cq(i, c) - U[c]);
    lam[static_cast<size_t>(i) * n + cell] = static_cast<R>(s * inv_rho);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const R lb = static_cast<R>(dl_db ? dl_db[c * n + cell] : 0.0);
#pragma unroll
    for (int i = 0; i < 7; ++i) lam[static_cast<size_t>(kQ + i * 3 + c) * n + cell] = lb;
  }
}

// ------------------------------------------------------------------ reductions
constexpr int kRedThreads = 256;
constexpr int kRedBlocksMax = 2048;

__device__ __forceinline__ void reduce_add(const NodeQ& q, double (&acc)[FLAME_NRED]) {
  const double u2 = q.U[0] * q.U[0] + q.U[1] * q.U[1] + q.U[2] * q.U[2];
  acc[0] += 0.5 * u2;
  acc[1] += 0.5 * (q.b[0] * q.b[0] + q.b[1] * q.b[1] + q.b[2] * q.b[2]);
  acc[2] += q.U[0] * q.b[0] + q.U[1] * q.b[1] + q.U[2] * q.b[2];
  acc[3] += q.J[0] * q.J[0] + q.J[1] * q.J[1] + q.J[2] * q.J[2];
  acc[4] = fmax(acc[4], fabs(q.divb));
  acc[5] += q.divb * q.divb;
  acc[6] = fmax(acc[6], sqrt(u2));
  acc[7] += (q.rho - 1.0) * (q.rho - 1.0);
  acc[8] += q.finite ? 0.0 : 1.0;
  acc[9] += q.rho;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    acc[10 + c] += q.rho * q.U[c];
    acc[13 + c] += q.B[c];
  }
}
// The block's partials from its threads' (tid of kRedThreads), by a fixed tree in sh.
__device__ __forceinline__ void reduce_block(const double (&acc)[FLAME_NRED], double (*sh)[kRedThreads], unsigned tid,
                                             double* partials) {
#pragma unroll
  for (int k = 0; k < FLAME_NRED; ++k) sh[k][tid] = acc[k];
  __syncthreads();
  for (unsigned s = kRedThreads / 2; s > 0; s >>= 1) {
    if (tid < s) {
      for (int k = 0; k < FLAME_NRED; ++k) {
        const double o = sh[k][tid + s];
        sh[k][tid] = (k == 4 || k == 6) ? fmax(sh[k][tid], o) : sh[k][tid] + o;
      }
    }
    __syncthreads();
  }
  if (tid < FLAME_NRED) partials[blockIdx.x * FLAME_NRED + tid] = sh[tid][0];
}

// Per-block partials: sums in every slot except 4 and 6 (maxima). Fixed grid and a fixed
// tree order make the result bitwise reproducible. Two blocks per CU at least: without that
// bound the FP64 instantiation takes 261 VGPRs (one wave per SIMD) and runs slower than with
// the few spills the bound costs.
template <typename S>
__global__ __launch_bounds__(kRedThreads, 2) void reduce_kernel(AuxArgs<S> a, double* partials) {
  double acc[FLAME_NRED] = {};
  const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
  for (size_t cell = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; cell < a.v.n; cell += stride) {
    int x, y, z;
    node_xyz(cell, a.v.nx, a.v.ny, x, y, z);
    reduce_add(node_quantities(a, x, y, z), acc);
  }
  __shared__ double sh[FLAME_NRED][kRedThreads];
  reduce_block(acc, sh, threadIdx.x, partials);
}

// Node fields (REDUCE false) or reductions of the curl-stencil route. A workgroup marches tiles of 64 x 4
// along z with b of four planes and of the ring around the tile in LDS, as the step does, so a node's
// magnetic populations are read once for the curls of its neighbours: reading them at each of the six
// neighbours took 84 more loads a node (192 x 160 x 176 FP32: fields 567 us, reductions 826). Every sum
// has the order of node_quantities. Bound by HBM and the ring's re-reads.
constexpr int kMarchRows = kRedThreads / 64;
struct FieldPtrs {
  double *rho, *u, *B, *J, *divb;
};
template <typename S, int FM, bool REDUCE>
__global__ __launch_bounds__(kRedThreads) void stencil_march_kernel(AuxArgs<S> a, int planes, uint32_t items, FieldPtrs o,
                                                                    double* partials) {
  using E = Enc<S>;
  constexpr Addr A = Addr::Global;
  constexpr int TX = 64, TY = kMarchRows;
  __shared__ double lds[4 * (TY + 2) * (TX + 2) * 3];
  static_assert(sizeof(lds) >= sizeof(double) * FLAME_NRED * kRedThreads, "the block tree reuses the tile's LDS");
  double(*sb)[TY + 2][TX + 2][3] = reinterpret_cast<double(*)[TY + 2][TX + 2][3]>(lds);
  const View<S>& v = a.v;
  const int nx = v.nx, ny = v.ny, nz = v.nz;
  const uint32_t plane = static_cast<uint32_t>(nx) * ny;
  const int lx = threadIdx.x % TX, ly = threadIdx.x / TX;
  const uint32_t gx = (nx + TX - 1) / TX, gy = (ny + TY - 1) / TY;
  double acc[FLAME_NRED] = {};
  for (uint32_t it = gridDim.x == items ? logical_index(items) : blockIdx.x; it < items; it += gridDim.x) {
    const int x0 = (it % gx) * TX, y0 = (it / gx % gy) * TY, z_begin = it / (gx * gy) * planes;
    const int w = min(TX, nx - x0), h = min(TY, ny - y0), z_end = min(nz, z_begin + planes);
    const bool active = lx < w && ly < h;
    const Rows rw(active ? x0 + lx : 0, active ? y0 + ly : 0, nx, ny);
    auto pull = [&](const Rows& r, const Planes& pl, int i, int c) {
      const uint32_t off = r.at(-xim(i, 0), -xim(i, 1)) + pl.at(-xim(i, 2));
      return static_cast<double>(ld<A>(v.G + static_cast<size_t>(i * 3 + c) * v.stride, off)) / E::mscale(i);
    };
    auto half_src = [&](uint32_t cell, int c) {
      return a.force_b ? 0.5 * static_cast<double>(a.force_b[static_cast<size_t>(c) * v.n + cell]) : 0.0;
    };
    // b of the node's own populations into slot; their trace of Lambda and finiteness
    auto own = [&](int slot, const Planes& pl, double& tr, bool& fin) {
      double g[kM];
#pragma unroll
      for (int i = 0; i < 7; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) g[i * 3 + c] = pull(rw, pl, i, c);
      fin = true;
#pragma unroll
      for (int q = 0; q < kM; ++q) fin = fin && isfinite(g[q]);
      double b[3], lam[3][3];
      magnetic_moments(g, b, lam);
      tr = lam[0][0] + lam[1][1] + lam[2][2];
      const uint32_t cell = rw.at(0, 0) + pl.at(0);
#pragma unroll
      for (int c = 0; c < 3; ++c) sb[slot][ly + 1][lx + 1][c] = a.force_b ? b[c] + half_src(cell, c) : b[c];
    };
    // the ring: y-neighbours enter through B_x and B_z, x-neighbours through B_y and B_z
    auto ring = [&](int slot, const Planes& pl) {
      for (int task = threadIdx.x; task < 2 * w + 2 * h; task += kRedThreads) {
        const bool side = task >= 2 * w;
        const int t = side ? task - 2 * w : task, len = side ? h : w, at = t < len ? t : t - len;
        const int rx = side ? (t < h ? -1 : w) : at, ry = side ? at : (t < w ? -1 : h);
        const Rows rr(wrap(x0 + rx, nx), wrap(y0 + ry, ny), nx, ny);
        const uint32_t cell = rr.at(0, 0) + pl.at(0);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int c = k == 1 ? 2 : side ? 1 : 0;
          double b = pull(rr, pl, 0, c);
#pragma unroll
          for (int i = 1; i < 7; ++i) b += pull(rr, pl, i, c);
          sb[slot][ry + 1][rx + 1][c] = a.force_b ? b + half_src(cell, c) : b;
        }
      }
    };
    double tr = 0, tr_next = 0;
    bool fin = true, fin_next = true;
    const Planes p0(z_begin, nz, plane);
    if (active) {
      own(0, Planes(wrap(z_begin - 1, nz), nz, plane), tr, fin);
      own(1, p0, tr_next, fin_next);
    }
    ring(1, p0);
    int prev = 0, cur = 1, next = 2, spare = 3;
    for (int z = z_begin; z < z_end; ++z) {
      const Planes pl(z, nz, plane), pn(wrap(z + 1, nz), nz, plane);
      const uint32_t cell = rw.at(0, 0) + pl.at(0);
      tr = tr_next;
      fin = fin_next;
      NodeQ q;
      if (active) own(next, pn, tr_next, fin_next);
      ring(next, pn);
      if (active) {
        double drho = 0, j[3] = {0, 0, 0};
#pragma unroll
        for (int i = 0; i < kQ; ++i) {
          const uint32_t off = FM == 0 ? cell : rw.at(-cq(i, 0), -cq(i, 1)) + pl.at(-cq(i, 2));
          const double f =
              static_cast<double>(ld<A>(v.F + static_cast<size_t>(FM == 1 ? oppq(i) : i) * v.stride, off)) / E::fscale(i);
          fin = fin && isfinite(f);
          drho += f;
#pragma unroll
          for (int c = 0; c < 3; ++c)
            if (cq(i, c) != 0) j[c] += cq(i, c) * f;
        }
        // an infinite population makes every component NaN, as the velocities of node_quantities that are 0
        // along it do (three operations here instead of 27: 0.5% of the reductions' time)
#pragma unroll
        for (int c = 0; c < 3; ++c) j[c] += 0.0 * drho;
        q.rho = 1.0 + drho;
        q.finite = fin;
        q.divb = -4.0 * a.omega_b * tr;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const double F = a.force_u ? static_cast<double>(a.force_u[static_cast<size_t>(c) * v.n + cell]) : 0.0;
          q.U[c] = (j[c] + 0.5 * F) / q.rho;
        }
      }
      __syncthreads();   // a slot is rewritten two planes after it was last read: one barrier a plane
      if (active) {
        const double(&P)[TY + 2][TX + 2][3] = sb[prev];
        const double(&C)[TY + 2][TX + 2][3] = sb[cur];
        const double(&N)[TY + 2][TX + 2][3] = sb[next];
        const int px = lx + 1, py = ly + 1;
        q.J[0] = 0.5 * (C[py + 1][px][2] - C[py - 1][px][2]) - 0.5 * (N[py][px][1] - P[py][px][1]);
        q.J[1] = 0.5 * (N[py][px][0] - P[py][px][0]) - 0.5 * (C[py][px + 1][2] - C[py][px - 1][2]);
        q.J[2] = 0.5 * (C[py][px + 1][1] - C[py][px - 1][1]) - 0.5 * (C[py + 1][px][0] - C[py - 1][px][0]);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          q.b[c] = C[py][px][c];
          q.B[c] = a.b0[c] + q.b[c];
        }
        if (REDUCE) {
          reduce_add(q, acc);
        } else {
          if (o.rho) o.rho[cell] = q.rho;
          if (o.divb) o.divb[cell] = q.divb;
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            if (o.u) o.u[c * v.n + cell] = q.U[c];
            if (o.B) o.B[c * v.n + cell] = q.B[c];
            if (o.J) o.J[c * v.n + cell] = q.J[c];
          }
        }
      }
      const int t = prev;
      prev = cur;
      cur = next;
      next = spare;
      spare = t;
    }
    __syncthreads();   // the next item, or the block tree, rewrites the LDS
  }
  if (REDUCE) reduce_block(acc, reinterpret_cast<double(*)[kRedThreads]>(lds), threadIdx.x, partials);
}

// Fixed-order merge of the block partials of reduce_kernel into the FLAME_NRED results: thread
// (g, k) runs over the blocks g, g + 64, ... in order for slot k (sums; maxima for slots 4 and 6), the
// 64 groups meet in a fixed tree, and the slot is normalised as flame_reduce documents (node
// averages, rms, plain sums and maxima). One thread per slot over all 2048 blocks took 700 us, as
// long as the reduction of 200^3 nodes; this takes 12.
constexpr int kMergeGroups = 64;
__global__ __launch_bounds__(kMergeGroups * FLAME_NRED) void reduce_merge_kernel(const double* partials, int blocks,
                                                                                 double n, double* out) {
  __shared__ double sh[kMergeGroups][FLAME_NRED];
  const int k = threadIdx.x % FLAME_NRED, g = threadIdx.x / FLAME_NRED;
  const bool max_slot = k == 4 || k == 6;
  double acc = 0.0;
#pragma unroll 8
  for (int b = g; b < blocks; b += kMergeGroups) {
    const double v = partials[static_cast<size_t>(b) * FLAME_NRED + k];
    acc = max_slot ? fmax(acc, v) : acc + v;
  }
  sh[g][k] = acc;
  __syncthreads();
  for (int s = kMergeGroups / 2; s > 0; s >>= 1) {
    if (g < s) sh[g][k] = max_slot ? fmax(sh[g][k], sh[g + s][k]) : sh[g][k] + sh[g + s][k];
    __syncthreads();
  }
  if (g > 0) return;
  acc = sh[0][k];
  if (k <= 3) acc = acc / n;
  else if (k == 5 || k == 7) acc = sqrt(acc / n);
  out[k] = acc;
}

}  // namespace flame

// Block partials of the allocation-free reductions (flame_reduce_noalloc): one row of FLAME_NRED
// doubles per reduction block, kRedBlocksMax rows (256 KiB). Each GPU the library runs on holds its
// own copy until the process ends; host code reaches it only through the address that
// hipGetSymbolAddress returns for the current device (see scratch_address), never by this name.
static __device__ __align__(256) double scratch[flame::kRedBlocksMax * FLAME_NRED];

namespace flame {

// ------------------------------------------------------------------ spectra
// Real fields that are transformed in place lie in rows of 2 (nx / 2 + 1) values, component arrays
// one after another.
__device__ __forceinline__ size_t padded_index(uint32_t cell, const GridShape& g, uint32_t pitch) {
  uint32_t x;
  const uint32_t row = div_by(cell, g.nx, x);
  return static_cast<size_t>(row) * pitch + x;
}

// Components first .. first + count - 1 of u (field 0) or B (field 1), each at dist doubles from
// the one before. The node's populations are read once for all of them.
template <typename S>
__global__ __launch_bounds__(256) void field_kernel(AuxArgs<S> a, GridShape shape, int field, int first, int count,
                                                    uint32_t pitch, size_t dist, double* out) {
  const size_t cell = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
  if (cell >= a.v.n) return;
  int x, y, z;
  node_xyz(cell, a.v.nx, a.v.ny, x, y, z);
  const View<S>& v = a.v;
  double r[3];
  if (field == 0) {
    double f[kQ];
    if (v.fmode == 0) view_fluid<0>(v, x, y, z, f);
    else if (v.fmode == 1) view_fluid<1>(v, x, y, z, f);
    else view_fluid<2>(v, x, y, z, f);
    double drho = 0, j[3] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
      drho += f[i];
#pragma unroll
      for (int c = 0; c < 3; ++c) j[c] += cq(i, c) * f[i];   // also where c is 0, as in node_quantities
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double F = a.force_u ? static_cast<double>(a.force_u[static_cast<size_t>(c) * v.n + cell]) : 0.0;
      r[c] = (j[c] + 0.5 * F) / (1.0 + drho);
    }
  } else {
#pragma unroll
    for (int c = 0; c < 3; ++c)
      r[c] = a.b0[c] + (v.gmode == 0   ? field_fluct_m<0>(a, c, x, y, z)
                        : v.gmode == 1 ? field_fluct_m<1>(a, c, x, y, z)
                                       : field_fluct_m<2>(a, c, x, y, z));
  }
  double* at = out + padded_index(static_cast<uint32_t>(cell), shape, pitch);
#pragma unroll
  for (int c = 0; c < 3; ++c)
    if (c >= first && c < first + count) at[static_cast<size_t>(c - first) * dist] = r[c];
}

constexpr int kSpecShellsMax = 4096;

__device__ __forceinline__ int signed_freq(int idx, int n) { return idx <= (n - 1) / 2 ? idx : idx - n; }

// Shell binning without atomics. A binning block is one wavefront; it visits pieces of 64
// consecutive k_x of one (k_y, k_z) row in the fixed order of a grid-stride loop. Along such a piece
// the shell never decreases, so the entries of one shell are neighbouring lanes: a segmented scan in
// a fixed tree leaves each shell's sum in its last lane, which adds it to the block's LDS bins (one
// lane per shell). The block partials are then merged in a fixed order (bin_merge_kernel). Every
// sum therefore has one order for a given grid, and spectra are bitwise reproducible. All components
// are summed at an entry before it is binned. (A pass over the shells present among the lanes, with a
// sum over the wavefront for each, took 472 us per component at 256^3; this takes 100 for three.)
constexpr int kBinThreads = 64;
constexpr int kBinBlocksMax = 4096;

// Pieces of a half spectrum of rows of nxh entries.
struct HalfShape {
  int nx, ny, nz, nxh;
  uint32_t pieces;        // per row
  uint32_t total;         // pieces over all rows: at most 2^31, the nodes of the largest grid
  size_t nh;              // entries
};

// The entry of this lane in piece t: its index, or none (shell -1) beyond the row's end.
struct BinEntry {
  size_t k;
  int kx, ky, kz, shell;
};
__device__ __forceinline__ BinEntry bin_entry(uint32_t t, const HalfShape& h) {
  const uint32_t row = t / h.pieces, piece = t - row * h.pieces;
  BinEntry e;
  e.kz = static_cast<int>(row / static_cast<uint32_t>(h.ny));
  e.ky = static_cast<int>(row) - e.kz * h.ny;
  e.kx = static_cast<int>(piece * kBinThreads + threadIdx.x);
  e.k = static_cast<size_t>(row) * h.nxh + e.kx;
  const double fx = e.kx, fy = signed_freq(e.ky, h.ny), fz = signed_freq(e.kz, h.nz);
  e.shell = e.kx < h.nxh ? static_cast<int>(floor(sqrt(fx * fx + fy * fy + fz * fz) + 0.5)) : -1;
  return e;
}

// Orders LDS accesses between the lanes of a binning block, which is one wavefront: a lane's add follows the
// clearing and the adds of other lanes to the same bin. (No instruction: the hardware keeps the order of one
// wavefront's LDS operations.)
static_assert(kBinThreads == 64, "a binning block is one wavefront");
__device__ __forceinline__ void bins_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ void bins_clear(double* bins, int count) {
  for (int s = threadIdx.x; s < count; s += kBinThreads) bins[s] = 0.0;
  bins_sync();
}

// Add v of every lane to bins[shell]; called by all 64 lanes together.
__device__ __forceinline__ void bin_piece(double* bins, int nshells, int shell, double v) {
  const int lane = threadIdx.x;
#pragma unroll
  for (int off = 1; off < kBinThreads; off <<= 1) {
    const double below = __shfl_up(v, off, kBinThreads);
    const int s = __shfl_up(shell, off, kBinThreads);
    if (lane >= off && s == shell) v += below;
  }
  const int next = __shfl_down(shell, 1, kBinThreads);
  if ((lane == kBinThreads - 1 || next != shell) && shell >= 0 && shell < nshells) bins[shell] += v;
  bins_sync();
}

// Block partials of the bins, one row of nshells per block; added to what is there unless first.
__device__ __forceinline__ void bins_out(const double* bins, int nshells, int first, double* partials) {
  for (int s = threadIdx.x; s < nshells; s += kBinThreads) {
    double& out = partials[static_cast<size_t>(blockIdx.x) * nshells + s];
    out = first ? bins[s] : out + bins[s];
  }
}

// Half-spectra (nz, ny, nx/2+1) of r2c transforms, comps of them; each entry stands for itself and,
// for 0 < kx < nx - kx, its conjugate mirror at -k (same shell). Each entry adds w |X|^2 norm2 to
// its shell: w = 1/2 for the energy spectrum; w = |q|^2, q_a = 2 pi k_a / n_a, for the
// dissipation spectrum (k2 set).
__global__ __launch_bounds__(kBinThreads) void shell_bin_kernel(const hipfftDoubleComplex* X, int comps, HalfShape h,
                                                                int nshells, double norm2, int k2, int first,
                                                                double* partials) {
  extern __shared__ double bins[];
  bins_clear(bins, nshells);
  for (uint32_t t = blockIdx.x; t < h.total; t += gridDim.x) {
    const BinEntry e = bin_entry(t, h);
    double v = 0.0;
    if (e.shell >= 0 && e.shell < nshells) {
      double p = 0.0;
      for (int c = 0; c < comps; ++c) {
        const hipfftDoubleComplex x = X[c * h.nh + e.k];
        p += x.x * x.x + x.y * x.y;
      }
      double w = 0.5;
      if (k2) {
        const double qx = (2.0 * M_PI / h.nx) * e.kx, qy = (2.0 * M_PI / h.ny) * signed_freq(e.ky, h.ny),
                     qz = (2.0 * M_PI / h.nz) * signed_freq(e.kz, h.nz);
        w = qx * qx + qy * qy + qz * qz;
      }
      v = ((e.kx == 0 || 2 * e.kx == h.nx) ? 1.0 : 2.0) * w * p * norm2;
    }
    bin_piece(bins, nshells, e.shell, v);
  }
  bins_out(bins, nshells, first, partials);
}

// out[t][s] = sum over blocks of partials[t][block][s] (terms t < gridDim.y): thread (g, s) runs
// over the blocks g, g + 64, ... in order, the 64 groups meet in a fixed tree (4096 blocks of 129 shells:
// 16 groups 79 us, 64 groups 20).
constexpr int kBinMergeShells = 16;
constexpr int kBinMergeGroups = 64;
__global__ __launch_bounds__(kBinMergeShells * kBinMergeGroups) void bin_merge_kernel(const double* partials, int blocks,
                                                                                      int nshells, double* out) {
  __shared__ double sh[kBinMergeGroups][kBinMergeShells];
  const int l = threadIdx.x % kBinMergeShells, g = threadIdx.x / kBinMergeShells;
  const int s = blockIdx.x * kBinMergeShells + l;
  const size_t t = blockIdx.y;
  double acc = 0.0;
  if (s < nshells) {
    const double* p = partials + t * blocks * nshells + s;
#pragma unroll 8
    for (int b = g; b < blocks; b += kBinMergeGroups) acc += p[static_cast<size_t>(b) * nshells];
  }
  sh[g][l] = acc;
  __syncthreads();
  for (int w = kBinMergeGroups / 2; w > 0; w >>= 1) {
    if (g < w) sh[g][l] += sh[g + w][l];
    __syncthreads();
  }
  if (g == 0 && s < nshells) out[t * nshells + s] = sh[0][l];
}

// ------------------------------------------------------------------ energy transfer
// Derivative wavenumber 2 pi k / n of the DFT index idx (signed), 0 on the Nyquist index of an
// even axis (that mode's derivative is not a real field).
__device__ __forceinline__ double deriv_q(int idx, int n) {
  return 2 * idx == n ? 0.0 : (2.0 * M_PI / n) * signed_freq(idx, n);
}

// Padded copies (rows of pitch values, dist apart) of three arrays of n nodes each: what the
// in-place transforms read.
__global__ __launch_bounds__(256) void pad_kernel(const double* src, GridShape g, uint32_t pitch, size_t dist, double* dst) {
  const uint32_t cell = blockIdx.x * 256u + threadIdx.x;
  if (cell >= g.n) return;
  double* at = dst + padded_index(cell, g, pitch);
#pragma unroll
  for (int c = 0; c < 3; ++c) at[c * dist] = src[static_cast<size_t>(c) * g.n + cell];
}

// out_a = i q_a X / ncell on the half spectrum for the axes first .. first + count - 1: the inverse
// real transform of out_a is the derivative along a of the field whose unnormalised forward
// transform is X.
__global__ __launch_bounds__(256) void spectral_derivative_kernel(const hipfftDoubleComplex* X, HalfShape h, Divisor row,
                                                                  Divisor rows, double inv_n, int first, int count,
                                                                  hipfftDoubleComplex* out) {
  const size_t k = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
  if (k >= h.nh) return;
  uint32_t kx, ky;
  const uint32_t r = div_by(static_cast<uint32_t>(k), row, kx);
  const uint32_t kz = div_by(r, rows, ky);
  const double q[3] = {deriv_q(kx, h.nx) * inv_n, deriv_q(ky, h.ny) * inv_n, deriv_q(kz, h.nz) * inv_n};
  const hipfftDoubleComplex x = X[k];
#pragma unroll
  for (int a = 0; a < 3; ++a)
    if (a >= first && a < first + count) out[(a - first) * h.nh + k] = make_hipDoubleComplex(-q[a] * x.y, q[a] * x.x);
}

// out = (first == 0 ? 0 : out) + sum over the count axes from first of U_a d_a, node by node, with d
// and out padded and U three arrays of n nodes.
__global__ __launch_bounds__(256) void advect_kernel(const double* U, const double* d, GridShape g, uint32_t pitch,
                                                     size_t dist, int first, int count, double* out) {
  const uint32_t cell = blockIdx.x * 256u + threadIdx.x;
  if (cell >= g.n) return;
  const size_t at = padded_index(cell, g, pitch);
  double s = first == 0 ? 0.0 : out[at];
  for (int a = 0; a < count; ++a) s += U[static_cast<size_t>(first + a) * g.n + cell] * d[a * dist + at];
  out[at] = s;
}

// Components first .. first + count - 1 of P x Q, padded, with P and Q three consecutive arrays of n nodes.
__global__ __launch_bounds__(256) void cross_kernel(const double* P, const double* Q, GridShape g, uint32_t pitch,
                                                    size_t dist, int first, int count, double* out) {
  const uint32_t cell = blockIdx.x * 256u + threadIdx.x;
  if (cell >= g.n) return;
  double p[3], q[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    p[c] = P[static_cast<size_t>(c) * g.n + cell];
    q[c] = Q[static_cast<size_t>(c) * g.n + cell];
  }
  double* at = out + padded_index(cell, g, pitch);
#pragma unroll
  for (int c = 0; c < 3; ++c)
    if (c >= first && c < first + count) at[(c - first) * dist] = p[(c + 1) % 3] * q[(c + 2) % 3] - p[(c + 2) % 3] * q[(c + 1) % 3];
}

// Per-block shell sums of a transfer summand over the half spectrum (entries with 0 < kx < nx - kx
// stand for their mirror too, whose summand is equal), summed over the components c0 .. c0 + count - 1
// that Y holds. With x set, sign Re[conj(X_c) Y_c] into partials; with induction set,
// induction times -Re[i Y_c (conj(B_hat) x q)_c] into ipartials, B_hat the three transforms in Bh. Added
// to what is there unless c0 is 0. Binned without atomics, as shell_bin_kernel.
__global__ __launch_bounds__(kBinThreads) void transfer_bin_kernel(const hipfftDoubleComplex* X, double sign,
                                                                   const hipfftDoubleComplex* Y,
                                                                   const hipfftDoubleComplex* Bh, double induction,
                                                                   int c0, int count, HalfShape h, int nshells,
                                                                   double norm2, double* partials, double* ipartials) {
  extern __shared__ double bins[];
  double* ibins = bins + (X ? nshells : 0);
  bins_clear(bins, (X ? nshells : 0) + (Bh ? nshells : 0));
  for (uint32_t t = blockIdx.x; t < h.total; t += gridDim.x) {
    const BinEntry e = bin_entry(t, h);
    double v = 0.0, w = 0.0;
    if (e.shell >= 0 && e.shell < nshells) {
      const double q[3] = {deriv_q(e.kx, h.nx), deriv_q(e.ky, h.ny), deriv_q(e.kz, h.nz)};
      hipfftDoubleComplex B[3];
      if (Bh)
        for (int c = 0; c < 3; ++c) B[c] = Bh[c * h.nh + e.k];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if (c < c0 || c >= c0 + count) continue;
        const hipfftDoubleComplex y = Y[(c - c0) * h.nh + e.k];
        if (X) {
          const hipfftDoubleComplex x = X[c * h.nh + e.k];
          v += x.x * y.x + x.y * y.y;
        }
        if (Bh) {
          // z = (conj(B_hat) x q)_c = conj(B_d) q_e - conj(B_e) q_d; -Re[i y z] = Im[y z]
          const int d = (c + 1) % 3, f = (c + 2) % 3;
          const double zr = B[d].x * q[f] - B[f].x * q[d];
          const double zi = -B[d].y * q[f] + B[f].y * q[d];
          w += y.x * zi + y.y * zr;
        }
      }
      const double mult = (e.kx == 0 || 2 * e.kx == h.nx) ? norm2 : 2.0 * norm2;
      v *= sign * mult;
      w *= induction * mult;
    }
    if (X) bin_piece(bins, nshells, e.shell, v);
    if (Bh) bin_piece(ibins, nshells, e.shell, w);
  }
  if (X) bins_out(bins, nshells, c0 == 0, partials);
  if (Bh) bins_out(ibins, nshells, c0 == 0, ipartials);
}

}  // namespace flame

using namespace flame;

// ====================================================================== host side
namespace {

thread_local std::string g_init_error;

flame_status fail(flame_ctx* c, flame_status code, const std::string& msg) {
  if (c) c->err = msg; else g_init_error = msg;
  return code;
}

#define FLAME_HIP(c, call)                                                        \
  do {                                                                            \
    hipError_t e_ = (call);                                                       \
    if (e_ != hipSuccess)                                                         \
      return fail((c), FLAME_E_HIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

std::string validate(const flame_params* p) {
  if (!p) return "params is NULL";
  if (p->nx < 1 || p->ny < 1 || p->nz < 1) return "grid sizes must be >= 1";
  if (p->jmode == FLAME_J_STENCIL && (p->nx < 3 || p->ny < 3 || p->nz < 3))
    return "the stencil current needs every grid size >= 3";
  const double cells = static_cast<double>(p->nx) * p->ny * p->nz;
  if (cells >= 1099511627776.0) return "grid too large (nx*ny*nz must be < 2^40)";
  if (p->nz > 65535) return "nz must be <= 65535";
  // kernels address each population and forcing array with 32-bit byte offsets: every array,
  // with its stride padding, must span at most 4 GiB (largest offset 4 GiB minus one value)
  const double vb = p->storage == FLAME_F64 ? 8.0 : p->storage == FLAME_F32 ? 4.0 : 2.0;
  const double fb = p->storage == FLAME_F64 ? 8.0 : 4.0;
  const bool forced = p->force_u || p->force_b;
  if (cells >= 4294967296.0 || static_cast<double>(population_stride(*p)) * vb > 4294967296.0 ||
      (forced && cells * fb > 4294967296.0))
    return "grid too large: each population / forcing array must fit in 4 GiB";
  if (!(p->nu > 0) || !isfinite(p->nu)) return "nu must be finite and > 0";
  if (!(p->eta > 0) || !isfinite(p->eta)) return "eta must be finite and > 0";
  if (!(p->d_i >= 0) || !isfinite(p->d_i)) return "d_i must be finite and >= 0";
  for (int i = 0; i < 3; ++i)
    if (!isfinite(p->b0[i])) return "b0 must be finite";
  if (p->storage != FLAME_F64 && p->storage != FLAME_F32 && p->storage != FLAME_F16)
    return "unknown storage";
  if (p->jmode != FLAME_J_MOMENT && p->jmode != FLAME_J_STENCIL) return "unknown jmode";
  if (p->layout != FLAME_LAYOUT_AB && p->layout != FLAME_LAYOUT_AA) return "unknown layout";
  if (p->collision != FLAME_COLLISION_CENTRAL && p->collision != FLAME_COLLISION_BGK) return "unknown collision";
  if (p->magnetic != FLAME_MAGNETIC_HALL && p->magnetic != FLAME_MAGNETIC_EMHD) return "unknown magnetic model";
  if (p->fluid_lattice != FLAME_FLUID_D3Q27 && p->fluid_lattice != FLAME_FLUID_D3Q19) return "unknown fluid lattice";
  if (p->magnetic_lattice != FLAME_MAGNETIC_D3Q7 && p->magnetic_lattice != FLAME_MAGNETIC_D3Q15 &&
      p->magnetic_lattice != FLAME_MAGNETIC_D3Q27)
    return "unknown magnetic lattice";
  return "";
}

// Valid parameters whose combination is not built ("" if it is).
std::string unsupported(const flame_params* p) {
  if (lattice_variant(*p) && p->jmode != FLAME_J_MOMENT)
    return "the lattice variants run the moment route of J only";
  if (p->fluid_lattice == FLAME_FLUID_D3Q19 && p->collision != FLAME_COLLISION_BGK)
    return "the central-moment collision is built on the D3Q27 fluid set; D3Q19 runs the BGK collision";
  return "";
}

size_t values_per_node(const flame_params& p) {
  const size_t one = static_cast<size_t>(fluid_count(p)) + 3 * static_cast<size_t>(mag_count(p));
  if (p.layout == FLAME_LAYOUT_AB) return 2 * one;
  return p.jmode == FLAME_J_STENCIL ? one + 3 * static_cast<size_t>(mag_count(p)) : one;
}

template <typename S>
View<S> make_view(const flame_ctx* c) {
  const SetPtrs s = set_ptrs(c);
  View<S> v;
  v.F = static_cast<const S*>(s.f_src);
  v.G = static_cast<const S*>(s.g_src);
  v.fmode = s.fluid_aa ? (c->parity == 1 ? 1 : 0) : 2;
  v.gmode = s.mag_aa ? (c->parity == 1 ? 1 : 0) : 2;
  v.nx = c->p.nx;
  v.ny = c->p.ny;
  v.nz = c->p.nz;
  v.n = c->n;
  v.stride = c->stride;
  return v;
}

template <typename S>
AuxArgs<S> make_aux(const flame_ctx* c) {
  using R = typename Enc<S>::R;
  AuxArgs<S> a;
  a.v = make_view<S>(c);
  a.force_u = static_cast<const R*>(c->p.force_u);
  a.force_b = static_cast<const R*>(c->p.force_b);
  for (int i = 0; i < 3; ++i) a.b0[i] = c->p.b0[i];
  a.alpha = c->p.d_i;
  a.omega_b = c->omega_b;
  a.emhd = c->p.magnetic == FLAME_MAGNETIC_EMHD;
  return a;
}

// Rest state for full-value copies; all zeros for deviation copies.
Rest make_rest(const flame_ctx* c, int32_t deviations) {
  Rest r;
  for (int i = 0; i < 27; ++i) r.f[i] = deviations ? 0.0 : c->frest[i];
  for (int i = 0; i < 3; ++i) r.b0[i] = deviations ? 0.0 : c->p.b0[i];
  return r;
}

Placement make_placement(const flame_ctx* c) {
  const SetPtrs s = set_ptrs(c);
  Placement at;
  at.fpull = !s.fluid_aa;
  at.gpull = !s.mag_aa;
  at.nx = c->p.nx;
  at.ny = c->p.ny;
  at.nz = c->p.nz;
  return at;
}

unsigned blocks_for(size_t n, int threads) { return static_cast<unsigned>((n + threads - 1) / threads); }

// Dispatch a callable templated on the storage type.
template <typename Fn>
hipError_t by_storage(const flame_ctx* c, Fn&& fn) {
  switch (c->p.storage) {
    case FLAME_F64: return fn(double{});
    case FLAME_F32: return fn(float{});
    default: return fn(_Float16{});
  }
}

__global__ void max_field_kernel(const double* b, double b0x, double b0y, double b0z, size_t n, double* out) {
  __shared__ double sh[256];
  double m = 0.0;
  for (size_t k = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; k < n;
       k += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const double x = b0x + b[k], y = b0y + b[n + k], z = b0z + b[2 * n + k];
    m = fmax(m, sqrt(x * x + y * y + z * z));
  }
  sh[threadIdx.x] = m;
  __syncthreads();
  for (unsigned s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = sh[0];
}

// Device address of this device's copy of the scratch array, looked up once per device (with that
// device current) and kept for the process.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
double* g_scratch_addr[kMaxDevices] = {};

hipError_t scratch_address(int device, double** out) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_addr[device]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_addr[device] = static_cast<double*>(ptr);
  }
  *out = g_scratch_addr[device];
  return hipSuccess;
}

// Lattice sound speed c_s = 1/sqrt(3): the flame_reduce guard on max |u|.
constexpr double kSoundSpeed = 0.57735026918962576;

// Node fields (partials null) or block partials of the stencil route; blocks returns the partials' rows.
hipError_t launch_stencil_march(const flame_ctx* c, const FieldPtrs& o, double* partials, int& blocks) {
  const uint32_t tiles = static_cast<uint32_t>((c->p.nx + 63) / 64) * ((c->p.ny + kMarchRows - 1) / kMarchRows);
  const int planes = march_planes(tiles, c->p.nz, static_cast<int64_t>(c->cus) * 4, 32);
  const uint32_t items = tiles * ((c->p.nz + planes - 1) / planes);
  blocks = static_cast<int>(partials ? std::min<uint32_t>(items, kRedBlocksMax) : items);
  return by_storage(c, [&](auto tag) {
    using S = decltype(tag);
    const AuxArgs<S> a = make_aux<S>(c);
    auto go = [&](auto mode) {
      constexpr int FM = decltype(mode)::value;
      if (partials)
        hipLaunchKernelGGL((stencil_march_kernel<S, FM, true>), dim3(blocks), dim3(kRedThreads), 0, c->stream, a, planes,
                           items, o, partials);
      else
        hipLaunchKernelGGL((stencil_march_kernel<S, FM, false>), dim3(blocks), dim3(kRedThreads), 0, c->stream, a, planes,
                           items, o, partials);
    };
    if (a.v.fmode == 0) go(std::integral_constant<int, 0>{});
    else if (a.v.fmode == 1) go(std::integral_constant<int, 1>{});
    else go(std::integral_constant<int, 2>{});
    return hipGetLastError();
  });
}

// Node fields of the current state, each array optional. Asynchronous.
hipError_t launch_moments(const flame_ctx* c, double* rho, double* u, double* b, double* j, double* divb) {
  if (lattice_variant(c->p)) return variant_launch_moments(c, rho, u, b, j, divb);
  if (c->p.jmode == FLAME_J_STENCIL) {
    int blocks;
    return launch_stencil_march(c, FieldPtrs{rho, u, b, j, divb}, nullptr, blocks);
  }
  return by_storage(c, [&](auto tag) {
    using S = decltype(tag);
    hipLaunchKernelGGL(moments_kernel<S>, dim3(blocks_for(c->n, 256)), dim3(256), 0, c->stream, make_aux<S>(c), rho, u, b,
                       j, divb);
    return hipGetLastError();
  });
}

// The reductions of the current state: block partials into partials (at most kRedBlocksMax x
// FLAME_NRED doubles), merged in a fixed order into out (FLAME_NRED doubles, device). Asynchronous.
hipError_t launch_reduce(const flame_ctx* c, double* partials, double* out) {
  int blocks = c->red_blocks;
  hipError_t e;
  if (lattice_variant(c->p)) {
    e = variant_launch_reduce(c, partials);
  } else if (c->p.jmode == FLAME_J_STENCIL) {
    e = launch_stencil_march(c, FieldPtrs{}, partials, blocks);
  } else {
    e = by_storage(c, [&](auto tag) {
      using S = decltype(tag);
      hipLaunchKernelGGL(reduce_kernel<S>, dim3(c->red_blocks), dim3(kRedThreads), 0, c->stream, make_aux<S>(c),
                         partials);
      return hipGetLastError();
    });
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(reduce_merge_kernel, dim3(1), dim3(kMergeGroups * FLAME_NRED), 0, c->stream, partials, blocks,
                     static_cast<double>(c->n), out);
  return hipGetLastError();
}

}  // namespace

namespace flame {
SetPtrs set_ptrs(const flame_ctx* c) {
  const size_t vb = value_bytes(c->p.storage);
  const size_t n = c->stride;
  const size_t nf = fluid_count(c->p), ng = 3 * static_cast<size_t>(mag_count(c->p));
  char* base = static_cast<char*>(c->storage);
  SetPtrs s{};
  if (c->p.layout == FLAME_LAYOUT_AB) {
    char* F0 = base;
    char* F1 = base + nf * n * vb;
    char* G0 = base + 2 * nf * n * vb;
    char* G1 = G0 + ng * n * vb;
    s.f_src = c->cur ? F1 : F0;
    s.f_dst = c->cur ? F0 : F1;
    s.g_src = c->cur ? G1 : G0;
    s.g_dst = c->cur ? G0 : G1;
    s.fluid_aa = false;
    s.mag_aa = false;
  } else {
    s.f_src = s.f_dst = base;
    s.fluid_aa = true;
    char* G0 = base + nf * n * vb;
    if (c->p.jmode == FLAME_J_STENCIL) {
      char* G1 = G0 + ng * n * vb;
      s.g_src = c->cur ? G1 : G0;
      s.g_dst = c->cur ? G0 : G1;
      s.mag_aa = false;
    } else {
      s.g_src = s.g_dst = G0;
      s.mag_aa = true;
    }
  }
  return s;
}
}  // namespace flame

extern "C" {

flame_status flame_rest_populations(const flame_params* p, double* f_rest, double* g_rest) {
  if (!p) return FLAME_E_INVAL;
  if (lattice_variant(*p)) {
    if (!validate(p).empty()) return FLAME_E_INVAL;
    variant_rest(*p, f_rest, g_rest);
    return FLAME_OK;
  }
  // f^mhd(0)(1, 0, b0) = w_i + (w_i / 2 c_s^4) M(b0) : (c c - c_s^2 I), M = |b0|^2/2 I - b0 b0,
  // with M : (c c - I/3) = |b0|^2/2 (|c|^2 - 1/3) - (b0 . c)^2
  const double* B0 = p->b0;
  const double b2 = B0[0] * B0[0] + B0[1] * B0[1] + B0[2] * B0[2];
  if (f_rest)
    for (int i = 0; i < 27; ++i) {
      const double cb = cq(i, 0) * B0[0] + cq(i, 1) * B0[1] + cq(i, 2) * B0[2];
      f_rest[i] = wq(i) + wq(i) * 4.5 * (0.5 * b2 * (speed2q(i) - 1.0 / 3.0) - cb * cb);
    }
  if (g_rest)
    for (int i = 0; i < 7; ++i)
      for (int c = 0; c < 3; ++c) g_rest[i * 3 + c] = wm(i) * B0[c];
  return FLAME_OK;
}

size_t flame_storage_bytes(const flame_params* p) {
  if (!validate(p).empty() || !unsupported(p).empty()) return 0;
  return values_per_node(*p) * value_bytes(p->storage) * population_stride(*p);
}

flame_status flame_init(const flame_params* p, const double* u, const double* b, const double* grad_u,
                        const double* grad_b, void* storage, size_t storage_bytes, void* hip_stream,
                        flame_ctx** out) {
  g_init_error.clear();
  if (!out) return fail(nullptr, FLAME_E_INVAL, "out is NULL");
  *out = nullptr;
  const std::string bad = validate(p);
  if (!bad.empty()) return fail(nullptr, FLAME_E_INVAL, bad);
  const std::string not_built = unsupported(p);
  if (!not_built.empty()) return fail(nullptr, FLAME_E_UNSUPPORTED, not_built);
  if (!u || !b) return fail(nullptr, FLAME_E_INVAL, "u and b must be given");
  if (!storage) return fail(nullptr, FLAME_E_INVAL, "storage is NULL");
  if (reinterpret_cast<uintptr_t>(storage) % 256 != 0) return fail(nullptr, FLAME_E_INVAL, "storage must be 256-byte aligned");
  const size_t need = flame_storage_bytes(p);
  if (storage_bytes < need)
    return fail(nullptr, FLAME_E_INVAL, "storage too small: need " + std::to_string(need) + " bytes");
  flame_ctx* c = new (std::nothrow) flame_ctx;
  if (!c) return fail(nullptr, FLAME_E_NOMEM, "context allocation failed");
  c->p = *p;
  c->stream = static_cast<hipStream_t>(hip_stream);
  c->n = static_cast<size_t>(p->nx) * p->ny * p->nz;
  c->stride = population_stride(*p);
  c->storage = storage;
  c->omega = 1.0 / (3.0 * p->nu + 0.5);
  c->omega_b = 1.0 / (4.0 * p->eta + 0.5);
  // launch-shape tuning (multiples of 64 threads per row block; any positive plane count)
  if (const char* v = getenv("FLAME_ZCHUNK_PLANES")) c->zchunk = std::max(0, atoi(v));
  if (const char* v = getenv("FLAME_ROW_THREADS")) c->row_tx = std::min(std::max(0, atoi(v)) / 64 * 64, kRowThreadsMax);
  if (const char* v = getenv("FLAME_GLOBAL_ADDRESSING")) c->global_addr = atoi(v) != 0;
  if (const char* v = getenv("FLAME_SPECTRAL_BATCH")) c->spec_batch = atoi(v) == 1 ? 1 : 0;
  const double* B0 = p->b0;
  flame_rest_populations(p, c->frest, nullptr);   // q <= 27 values
  auto bail = [&](flame_status code) {
    g_init_error = c->err;
    delete c;
    return code;
  };
  if (hipGetDevice(&c->device) != hipSuccess) {
    c->err = "hipGetDevice failed (no HIP device?)";
    return bail(FLAME_E_HIP);
  }
  if (hipDeviceGetAttribute(&c->cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess) {
    c->err = "hipDeviceGetAttribute failed";
    return bail(FLAME_E_HIP);
  }
  {
    const hipError_t e = scratch_address(c->device, &c->scratch);
    if (e != hipSuccess) {
      c->err = std::string("hipGetSymbolAddress of the reduction scratch: ") + hipGetErrorString(e);
      return bail(FLAME_E_HIP);
    }
  }
  c->red_blocks = static_cast<int>(std::min<size_t>(kRedBlocksMax, blocks_for(c->n, kRedThreads)));
  // block partials of the reductions plus one row for their merged results
  if (hipMalloc(&c->red_partials, sizeof(double) * FLAME_NRED * (kRedBlocksMax + 1)) != hipSuccess) {
    c->err = "hipMalloc of reduction scratch failed";
    return bail(FLAME_E_NOMEM);
  }
  // initial state into the canonical slots of copy 0
  const SetPtrs s = set_ptrs(c);
  hipError_t e = lattice_variant(*p) ? variant_launch_init(c, u, b, grad_u, grad_b) : by_storage(c, [&](auto tag) {
    using S = decltype(tag);
    using R = typename Enc<S>::R;
    InitArgs<S> a;
    a.F = static_cast<S*>(s.f_src);
    a.G = static_cast<S*>(s.g_src);
    a.u = u;
    a.b = b;
    a.gu = grad_u;
    a.gb = grad_b;
    a.force_u = static_cast<const R*>(p->force_u);
    a.force_b = static_cast<const R*>(p->force_b);
    for (int i = 0; i < 3; ++i) a.b0[i] = B0[i];
    a.omega = c->omega;
    a.omega_b = c->omega_b;
    a.alpha = p->d_i;
    a.noneq = p->init_noneq;
    a.emhd = p->magnetic == FLAME_MAGNETIC_EMHD;
    a.nx = p->nx;
    a.ny = p->ny;
    a.nz = p->nz;
    a.n = c->n;
    a.stride = c->stride;
    a.at = make_placement(c);
    hipLaunchKernelGGL(init_kernel<S>, dim3(blocks_for(c->n, 256)), dim3(256), 0, c->stream, a);
    return hipGetLastError();
  });
  if (e != hipSuccess) {
    c->err = std::string("init kernel: ") + hipGetErrorString(e);
    return bail(FLAME_E_HIP);
  }
  // advisory CFL number from max |B| of the initial field
  const int mb = static_cast<int>(std::min<size_t>(1024, blocks_for(c->n, 256)));
  hipLaunchKernelGGL(max_field_kernel, dim3(mb), dim3(256), 0, c->stream, b, B0[0], B0[1], B0[2], c->n,
                     c->red_partials);
  double host[1024];
  e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(host, c->red_partials, sizeof(double) * mb, hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) {
    c->err = std::string("initial field maximum: ") + hipGetErrorString(e);
    return bail(FLAME_E_HIP);
  }
  double bmax = 0;
  for (int i = 0; i < mb; ++i) bmax = std::max(bmax, host[i]);
  c->cfl = M_PI * p->d_i * bmax;
  *out = c;
  return c->cfl > 1.0 ? FLAME_W_CFL : FLAME_OK;
}

flame_status flame_step(flame_ctx* c, int64_t nsteps) {
  if (!c) return FLAME_E_INVAL;
  if (nsteps < 0) return fail(c, FLAME_E_INVAL, "nsteps must be >= 0");
  const bool two_f = c->p.layout == FLAME_LAYOUT_AB;
  const bool two_g = mag_two_lattice(c->p);
  for (int64_t s = 0; s < nsteps; ++s) {
    const SetPtrs ptr = set_ptrs(c);
    hipError_t e = launch_step(c, ptr, c->stride, nullptr);
    if (e != hipSuccess) return fail(c, FLAME_E_HIP, std::string("step kernel: ") + hipGetErrorString(e));
    if (two_f || two_g) c->cur ^= 1;
    if (!two_f || !two_g) c->parity ^= 1;
    c->steps += 1;
  }
  return FLAME_OK;
}

flame_status flame_moments(flame_ctx* c, double* rho, double* u, double* b, double* j, double* divb) {
  if (!c) return FLAME_E_INVAL;
  const hipError_t e = launch_moments(c, rho, u, b, j, divb);
  if (e != hipSuccess) return fail(c, FLAME_E_HIP, std::string("moments kernel: ") + hipGetErrorString(e));
  return FLAME_OK;
}

flame_status flame_reduce(flame_ctx* c, double* out) {
  if (!c || !out) return c ? fail(c, FLAME_E_INVAL, "out is NULL") : FLAME_E_INVAL;
  // block partials, then the merged results behind them in the same scratch
  double* merged = c->red_partials + static_cast<size_t>(kRedBlocksMax) * FLAME_NRED;
  hipError_t e = launch_reduce(c, c->red_partials, merged);
  if (e != hipSuccess) return fail(c, FLAME_E_HIP, std::string("reduce kernel: ") + hipGetErrorString(e));
  FLAME_HIP(c, hipMemcpyAsync(out, merged, sizeof(double) * FLAME_NRED, hipMemcpyDeviceToHost, c->stream));
  FLAME_HIP(c, hipStreamSynchronize(c->stream));
  if (out[8] > 0) return fail(c, FLAME_E_NONFINITE, "non-finite populations at " + std::to_string(out[8]) + " nodes");
  if (out[6] >= kSoundSpeed)
    return fail(c, FLAME_E_UNSTABLE, "max |u| = " + std::to_string(out[6]) + " reached the lattice sound speed");
  return FLAME_OK;
}

flame_status flame_reduce_noalloc(flame_ctx* c, double* out) {
  if (!c || !out) return c ? fail(c, FLAME_E_INVAL, "out is NULL") : FLAME_E_INVAL;
  if (!c->scratch) return fail(c, FLAME_E_HIP, "the reduction scratch of this device was not found at init");
  if (c->red_blocks < 1 || c->red_blocks > kRedBlocksMax)
    return fail(c, FLAME_E_INVAL, "reduction needs " + std::to_string(c->red_blocks) +
                                      " block partials; the static scratch holds " + std::to_string(kRedBlocksMax));
  const hipError_t e = launch_reduce(c, c->scratch, out);
  if (e != hipSuccess) return fail(c, FLAME_E_HIP, std::string("reduce kernel: ") + hipGetErrorString(e));
  return FLAME_OK;
}

}  // extern "C"

namespace {

HalfShape half_shape(const flame_ctx* c) {
  HalfShape h;
  h.nx = c->p.nx;
  h.ny = c->p.ny;
  h.nz = c->p.nz;
  h.nxh = c->p.nx / 2 + 1;
  h.pieces = static_cast<uint32_t>((h.nxh + kBinThreads - 1) / kBinThreads);
  const size_t rows = static_cast<size_t>(h.ny) * h.nz;
  h.total = static_cast<uint32_t>(rows * h.pieces);
  h.nh = rows * h.nxh;
  return h;
}

// Device memory that a context keeps: at least count elements in ptr, which holds have.
template <typename T>
bool keep_at_least(T*& ptr, size_t& have, size_t count) {
  if (ptr && have >= count) return true;
  if (ptr) (void)hipFree(ptr);
  ptr = nullptr;
  have = 0;
  if (hipMalloc(&ptr, sizeof(T) * count) != hipSuccess) {
    ptr = nullptr;
    (void)hipGetLastError();  // clear the allocation error so later launch checks do not see it
    return false;
  }
  have = count;
  return true;
}

// Device memory that a context keeps between calls for the fields of a diagnostic: what is larger goes by
// one component at a time (the transforms) or is released at the end of the call (the energy transfer).
constexpr size_t kKeepBytes = size_t(4) << 30;

// A plan without a work area of its own; work returns the bytes that it needs.
bool make_plan(flame_ctx* c, hipfftHandle& plan, bool& ok, hipfftType type, size_t& work) {
  if (ok) return true;
  int n[3] = {c->p.nz, c->p.ny, c->p.nx};
  const int nxh = c->p.nx / 2 + 1;
  int real[3] = {c->p.nz, c->p.ny, 2 * nxh}, half[3] = {c->p.nz, c->p.ny, nxh};
  const bool many = c->spec_batch > 1;     // the distances only count then, and fit in an int (kKeepBytes)
  const int dist = many ? static_cast<int>(half_shape(c).nh) : 1, rdist = many ? 2 * dist : 1;
  const bool fwd = type == HIPFFT_D2Z;
  if (hipfftCreate(&plan) != HIPFFT_SUCCESS) return false;
  // a plan counts as made only once it runs on the context's stream
  ok = hipfftSetAutoAllocation(plan, 0) == HIPFFT_SUCCESS &&
       hipfftMakePlanMany(plan, 3, n, fwd ? real : half, 1, fwd ? rdist : dist, fwd ? half : real, 1, fwd ? dist : rdist,
                          type, c->spec_batch, &work) == HIPFFT_SUCCESS &&
       hipfftSetStream(plan, c->stream) == HIPFFT_SUCCESS;
  if (!ok) hipfftDestroy(plan);
  return ok;
}

// Release what the transforms of three components hold and go on with one.
void one_component(flame_ctx* c) {
  if (c->plan_ok) hipfftDestroy(c->plan);
  if (c->plan_inv_ok) hipfftDestroy(c->plan_inv);
  c->plan_ok = c->plan_inv_ok = false;
  c->plan_work = c->plan_inv_work = 0;
  if (c->spec_work) (void)hipFree(c->spec_work);
  if (c->fft_work) (void)hipFree(c->fft_work);
  c->spec_work = nullptr;
  c->fft_work = nullptr;
  c->spec_work_size = c->fft_work_size = 0;
  c->spec_batch = 1;
  (void)hipGetLastError();  // clear an allocation error so later launch checks do not see it
}

// Workspace of the in-place transforms: three components at once (one batched transform, one pass over
// the populations; 64^3 22 us against 3 x 12, from 256^3 on as fast as three), or one where three with the
// plans' work area (none, or one to four times as much again, by the prime factors and the size of the
// grid) are more than is kept, or where the memory for three (with the transfer values of transfer_work
// that the call needs) is not there.
flame_status spectral_setup(flame_ctx* c, int blocks, int terms, int nshells, bool inverse, size_t transfer) {
  const size_t nh = half_shape(c).nh;
  if (c->spec_batch == 0) c->spec_batch = 3 * nh * sizeof(hipfftDoubleComplex) <= kKeepBytes ? 3 : 1;
  for (;;) {
    const bool planned = make_plan(c, c->plan, c->plan_ok, HIPFFT_D2Z, c->plan_work) &&
                         (!inverse || make_plan(c, c->plan_inv, c->plan_inv_ok, HIPFFT_Z2D, c->plan_inv_work));
    const size_t work = std::max(c->plan_work, c->plan_inv_work);
    const bool kept = c->spec_batch == 1 || 3 * nh * sizeof(hipfftDoubleComplex) + work <= kKeepBytes;
    // block partials plus one row for their merged sums, per term
    const bool memory =
        planned && kept && keep_at_least(c->spec_work, c->spec_work_size, c->spec_batch * nh) &&
        (work == 0 || keep_at_least(c->fft_work, c->fft_work_size, work)) &&
        keep_at_least(c->spec_partials, c->spec_partials_size, static_cast<size_t>(terms) * (blocks + 1) * nshells) &&
        (transfer == 0 || keep_at_least(c->transfer_work, c->transfer_size, transfer));
    if (memory && (work == 0 || (hipfftSetWorkArea(c->plan, c->fft_work) == HIPFFT_SUCCESS &&
                                 (!c->plan_inv_ok || hipfftSetWorkArea(c->plan_inv, c->fft_work) == HIPFFT_SUCCESS))))
      return FLAME_OK;
    if (c->spec_batch == 1)
      return !planned || memory
                 ? fail(c, FLAME_E_HIP, "transform plan failed")
                 : fail(c, FLAME_E_NOMEM, transfer ? "energy transfer: device workspace" : "spectrum: device workspace");
    one_component(c);
  }
}

// Fewer blocks for many shells: the block partials stay within 64 MiB a term.
int bin_blocks(const HalfShape& h, int nshells) {
  const uint32_t most = std::min<uint32_t>(kBinBlocksMax, (uint32_t(8) << 20) / static_cast<uint32_t>(nshells));
  return static_cast<int>(std::min(most, h.total));
}

// Merge the block partials of the terms and copy the sums to the host.
hipError_t merged_bins(flame_ctx* c, int blocks, int terms, int nshells, double* host) {
  double* merged = c->spec_partials + static_cast<size_t>(terms) * blocks * nshells;
  hipLaunchKernelGGL(bin_merge_kernel, dim3((nshells + kBinMergeShells - 1) / kBinMergeShells, terms),
                     dim3(kBinMergeShells * kBinMergeGroups), 0, c->stream, c->spec_partials, blocks, nshells, merged);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess)
    e = hipMemcpyAsync(host, merged, sizeof(double) * terms * nshells, hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  return e;
}

// Energy (k2 = 0) or dissipation (k2 = 1) shell spectrum of u or B, summed over components.
flame_status shell_spectrum(flame_ctx* c, int32_t field, int32_t nshells, int k2, double* e_k) {
  if (!c) return FLAME_E_INVAL;
  if (field != 0 && field != 1) return fail(c, FLAME_E_INVAL, "field must be 0 (u) or 1 (B)");
  if (nshells < 1 || nshells > kSpecShellsMax) return fail(c, FLAME_E_INVAL, "nshells out of range");
  if (!e_k) return fail(c, FLAME_E_INVAL, "e_k is NULL");
  const HalfShape h = half_shape(c);
  const int blocks = bin_blocks(h, nshells);
  const flame_status ready = spectral_setup(c, blocks, 1, nshells, false, 0);
  if (ready != FLAME_OK) return ready;
  for (int s = 0; s < nshells; ++s) e_k[s] = 0.0;
  const double norm2 = 1.0 / (static_cast<double>(c->n) * static_cast<double>(c->n));
  const uint32_t pitch = 2 * static_cast<uint32_t>(h.nxh);
  double* real = reinterpret_cast<double*>(c->spec_work);
  for (int c0 = 0; c0 < 3; c0 += c->spec_batch) {
    hipError_t e = lattice_variant(c->p)
                       ? variant_launch_components(c, field, c0, c->spec_batch, pitch, 2 * h.nh, real)
                       : by_storage(c, [&](auto tag) {
      using S = decltype(tag);
      hipLaunchKernelGGL(field_kernel<S>, dim3(blocks_for(c->n, 256)), dim3(256), 0, c->stream, make_aux<S>(c),
                         grid_shape(c->p, 256), field, c0, c->spec_batch, pitch, 2 * h.nh, real);
      return hipGetLastError();
    });
    if (e != hipSuccess) return fail(c, FLAME_E_HIP, std::string("field kernel: ") + hipGetErrorString(e));
    if (hipfftExecD2Z(c->plan, real, c->spec_work) != HIPFFT_SUCCESS)
      return fail(c, FLAME_E_HIP, "hipfftExecD2Z failed");
    hipLaunchKernelGGL(shell_bin_kernel, dim3(blocks), dim3(kBinThreads), sizeof(double) * nshells, c->stream,
                       c->spec_work, c->spec_batch, h, nshells, norm2, k2, c0 == 0 ? 1 : 0, c->spec_partials);
    e = hipGetLastError();
    if (e != hipSuccess) return fail(c, FLAME_E_HIP, std::string("spectrum: ") + hipGetErrorString(e));
  }
  std::vector<double> host(static_cast<size_t>(nshells));
  const hipError_t e = merged_bins(c, blocks, 1, nshells, host.data());
  if (e != hipSuccess) return fail(c, FLAME_E_HIP, std::string("spectrum: ") + hipGetErrorString(e));
  for (int s = 0; s < nshells; ++s) e_k[s] = host[s];
  return FLAME_OK;
}

}  // namespace

extern "C" {

flame_status flame_spectrum(flame_ctx* c, int32_t field, int32_t nshells, double* e_k) {
  return shell_spectrum(c, field, nshells, 0, e_k);
}

flame_status flame_dissipation_spectrum(flame_ctx* c, int32_t field, int32_t nshells, double* d_k) {
  return shell_spectrum(c, field, nshells, 1, d_k);
}

}  // extern "C"

namespace {

// Node fields and transforms of the energy transfer (120 bytes a node), kept by the context up to
// kKeepBytes (330^3) and else released at the end of the call: allocating and freeing them took 30 ms of a
// 37 ms call at 192^3.
struct TransferRelease {
  flame_ctx* c;
  ~TransferRelease() {
    if (!c->transfer_work || c->transfer_size * sizeof(hipfftDoubleComplex) <= kKeepBytes) return;
    (void)hipStreamSynchronize(c->stream);   // work queued on an error path may still use it
    (void)hipFree(c->transfer_work);
    c->transfer_work = nullptr;
    c->transfer_size = 0;
  }
};

flame_status energy_transfer(flame_ctx* c, int32_t nshells, double* t_adv, double* t_lor, double* t_ind,
                             double* t_hall) {
  if (!c) return FLAME_E_INVAL;
  if (nshells < 1 || nshells > kSpecShellsMax) return fail(c, FLAME_E_INVAL, "nshells out of range");
  if (!t_adv || !t_lor || !t_ind) return fail(c, FLAME_E_INVAL, "an output array is NULL");
  const size_t n = c->n;
  const HalfShape h = half_shape(c);
  const GridShape g = grid_shape(c->p, 256);
  const uint32_t pitch = 2 * static_cast<uint32_t>(h.nxh);
  const size_t nh = h.nh, dist = 2 * nh;
  const int blocks = bin_blocks(h, nshells), terms = t_hall ? 4 : 3;
  // u_hat(3), B_hat(3), then the real fields U(3), B(3), J(3) (in units of a complex value)
  const size_t field3 = (3 * n + 1) / 2;
  TransferRelease release{c};
  const flame_status ready =
      spectral_setup(c, blocks, terms, nshells, true, 6 * nh + std::max(3 * field3, field3 + 3 * nh));
  if (ready != FLAME_OK) return ready;
  const int nb = c->spec_batch;
  hipfftDoubleComplex* Uh = c->transfer_work;
  hipfftDoubleComplex* Bh = Uh + 3 * nh;
  hipfftDoubleComplex* base = Uh + 6 * nh;
  double* U = reinterpret_cast<double*>(base);
  double* B = reinterpret_cast<double*>(base + field3);
  double* J = reinterpret_cast<double*>(base + 2 * field3);
  hipfftDoubleComplex* Ah = base + field3;      // the advection term, where B and J were
  hipfftDoubleComplex* spec = c->spec_work;     // nb components
  double* real = reinterpret_cast<double*>(spec);
  const unsigned gn = blocks_for(n, 256), gh = blocks_for(nh, 256);
  const hipError_t e = launch_moments(c, nullptr, U, B, J, nullptr);
  if (e != hipSuccess) return fail(c, FLAME_E_HIP, std::string("energy transfer fields: ") + hipGetErrorString(e));
  bool ok = true;
  auto launched = [&] { return ok = ok && hipGetLastError() == hipSuccess; };
  auto forward = [&](hipfftDoubleComplex* x) {
    return ok = ok && hipfftExecD2Z(c->plan, reinterpret_cast<double*>(x), x) == HIPFFT_SUCCESS;
  };
  const double norm2 = 1.0 / (static_cast<double>(n) * static_cast<double>(n));
  double* part[4];
  for (int t = 0; t < 4; ++t) part[t] = c->spec_partials + static_cast<size_t>(t) * blocks * nshells;
  auto bin = [&](const hipfftDoubleComplex* X, double sign, const hipfftDoubleComplex* Y, const hipfftDoubleComplex* Bx,
                 double induction, int c0, double* p, double* ip) {
    hipLaunchKernelGGL(transfer_bin_kernel, dim3(blocks), dim3(kBinThreads),
                       sizeof(double) * nshells * ((X ? 1 : 0) + (Bx ? 1 : 0)), c->stream, X, sign, Y, Bx, induction, c0,
                       nb, h, nshells, norm2, p, ip);
    return launched();
  };
  hipLaunchKernelGGL(pad_kernel, dim3(gn), dim3(256), 0, c->stream, U, g, pitch, dist, reinterpret_cast<double*>(Uh));
  launched();
  hipLaunchKernelGGL(pad_kernel, dim3(gn), dim3(256), 0, c->stream, B, g, pitch, dist, reinterpret_cast<double*>(Bh));
  launched();
  for (int b = 0; b < 6 && ok; b += nb) forward(Uh + b * nh);
  for (int b = 0; b < 3 && ok; b += nb) {
    // induction: (U x B)_b, binned against conj(B_hat) x q
    hipLaunchKernelGGL(cross_kernel, dim3(gn), dim3(256), 0, c->stream, U, B, g, pitch, dist, b, nb, real);
    launched() && forward(spec) && bin(nullptr, 0.0, spec, Bh, 1.0, b, nullptr, part[2]);
    // Lorentz force (J x B)_b; the Hall term takes the same transform against conj(B_hat) x q. Both
    // bins in one block need twice the LDS, which fits up to the largest shell count.
    if (!ok) break;
    hipLaunchKernelGGL(cross_kernel, dim3(gn), dim3(256), 0, c->stream, J, B, g, pitch, dist, b, nb, real);
    launched() && forward(spec) &&
        bin(Uh, -1.0, spec, t_hall ? Bh : nullptr, t_hall ? -c->p.d_i : 0.0, b, part[1], t_hall ? part[3] : nullptr);
  }
  // (U . grad) U_b, with grad U_b from the inverse transforms of i q_a u_hat_b
  for (int b = 0; b < 3 && ok; ++b)
    for (int a = 0; a < 3 && ok; a += nb) {
      hipLaunchKernelGGL(spectral_derivative_kernel, dim3(gh), dim3(256), 0, c->stream, Uh + b * nh, h, divisor(h.nxh),
                         divisor(h.ny), 1.0 / static_cast<double>(n), a, nb, spec);
      if (!launched()) break;
      ok = hipfftExecZ2D(c->plan_inv, spec, real) == HIPFFT_SUCCESS;
      if (!ok) break;
      hipLaunchKernelGGL(advect_kernel, dim3(gn), dim3(256), 0, c->stream, U, real, g, pitch, dist, a, nb,
                         reinterpret_cast<double*>(Ah + b * nh));
      launched();
    }
  for (int b = 0; b < 3 && ok; b += nb) forward(Ah + b * nh) && bin(Uh, 1.0, Ah + b * nh, nullptr, 0.0, b, part[0], nullptr);
  std::vector<double> host(static_cast<size_t>(terms) * nshells);
  if (ok) ok = merged_bins(c, blocks, terms, nshells, host.data()) == hipSuccess;
  if (!ok) {
    const hipError_t last = hipGetLastError();
    return fail(c, FLAME_E_HIP, std::string("energy transfer: a transform, copy or kernel launch failed (") +
                                    hipGetErrorString(last) + ")");
  }
  double* outs[4] = {t_adv, t_lor, t_ind, t_hall};
  for (int t = 0; t < terms; ++t)
    for (int s = 0; s < nshells; ++s) outs[t][s] = host[static_cast<size_t>(t) * nshells + s];
  return FLAME_OK;
}

}  // namespace

extern "C" {

flame_status flame_energy_transfer(flame_ctx* c, int32_t nshells, double* t_adv, double* t_lor, double* t_ind,
                                   double* t_hall) {
  return energy_transfer(c, nshells, t_adv, t_lor, t_ind, t_hall);
}

flame_status flame_get_populations(flame_ctx* c, double* dst, int32_t deviations) {
  if (!c || !dst) return c ? fail(c, FLAME_E_INVAL, "dst is NULL") : FLAME_E_INVAL;
  hipError_t e = lattice_variant(c->p) ? variant_launch_get(c, deviations, dst) : by_storage(c, [&](auto tag) {
    using S = decltype(tag);
    hipLaunchKernelGGL(get_kernel<S>, dim3(blocks_for(c->n, 256)), dim3(256), 0, c->stream, make_view<S>(c),
                       make_rest(c, deviations), dst);
    return hipGetLastError();
  });
  if (e != hipSuccess) return fail(c, FLAME_E_HIP, std::string("get kernel: ") + hipGetErrorString(e));
  return FLAME_OK;
}

flame_status flame_set_populations(flame_ctx* c, const double* src, int32_t deviations) {
  if (!c || !src) return c ? fail(c, FLAME_E_INVAL, "src is NULL") : FLAME_E_INVAL;
  c->cur = 0;
  c->parity = 0;
  c->steps = 0;
  const SetPtrs s = set_ptrs(c);
  hipError_t e = lattice_variant(c->p) ? variant_launch_set(c, deviations, src) : by_storage(c, [&](auto tag) {
    using S = decltype(tag);
    hipLaunchKernelGGL(set_kernel<S>, dim3(blocks_for(c->n, 256)), dim3(256), 0, c->stream,
                       static_cast<S*>(s.f_src), static_cast<S*>(s.g_src), c->n, c->stride, make_placement(c),
                       make_rest(c, deviations), src);
    return hipGetLastError();
  });
  if (e != hipSuccess) return fail(c, FLAME_E_HIP, std::string("set kernel: ") + hipGetErrorString(e));
  return FLAME_OK;
}

flame_status flame_gather(flame_ctx* c, const int64_t* cells, int64_t n, double* out, int32_t deviations) {
  if (!c) return FLAME_E_INVAL;
  if (n < 0 || (n > 0 && (!cells || !out))) return fail(c, FLAME_E_INVAL, "bad gather arguments");
  if (n == 0) return FLAME_OK;
  hipError_t e = lattice_variant(c->p) ? variant_launch_gather(c, deviations, cells, n, out) : by_storage(c, [&](auto tag) {
    using S = decltype(tag);
    hipLaunchKernelGGL(gather_kernel<S>, dim3(blocks_for(static_cast<size_t>(n), 256)), dim3(256), 0, c->stream,
                       make_view<S>(c), make_rest(c, deviations), cells, n, out);
    return hipGetLastError();
  });
  if (e != hipSuccess) return fail(c, FLAME_E_HIP, std::string("gather kernel: ") + hipGetErrorString(e));
  return FLAME_OK;
}

size_t flame_trace_bytes(const flame_ctx* c) {
  return c && reverse_mode_built(c->p) ? 48 * c->n * value_bytes(c->p.storage) : 0;
}

flame_status flame_trace_export(flame_ctx* c, void* lat) {
  if (!c) return FLAME_E_INVAL;
  if (c->p.layout != FLAME_LAYOUT_AA || c->p.jmode != FLAME_J_MOMENT)
    return fail(c, FLAME_E_UNSUPPORTED, "trace export is available on the moment route with the AA layout only");
  if (!reverse_mode_built(c->p))
    return fail(c, FLAME_E_UNSUPPORTED, "reverse mode is built for the paper's model and velocity sets only");
  if (!lat) return fail(c, FLAME_E_INVAL, "lat is NULL");
  hipError_t e = by_storage(c, [&](auto tag) {
    using S = decltype(tag);
    const SetPtrs p = set_ptrs(c);
    const S* F = static_cast<const S*>(p.f_src);
    const S* G = static_cast<const S*>(p.g_src);
    const GridShape g = grid_shape(c->p, row_threads(c->p.nx));
    if (c->parity == 0)
      hipLaunchKernelGGL((export_kernel<S, 0>), dim3(g.blocks), dim3(g.threads), 0, c->stream, F, G, c->stride, g, c->n,
                         static_cast<S*>(lat));
    else
      hipLaunchKernelGGL((export_kernel<S, 1>), dim3(g.blocks), dim3(g.threads), 0, c->stream, F, G, c->stride, g, c->n,
                         static_cast<S*>(lat));
    return hipGetLastError();
  });
  if (e != hipSuccess) return fail(c, FLAME_E_HIP, std::string("export kernel: ") + hipGetErrorString(e));
  return FLAME_OK;
}

flame_status flame_adjoint_fields(flame_ctx* c, const double* dl_du, const double* dl_db, void* lam) {
  if (!c) return FLAME_E_INVAL;
  if (!reverse_mode_built(c->p))
    return fail(c, FLAME_E_UNSUPPORTED, "reverse mode is built for the paper's model and velocity sets only");
  if (!lam) return fail(c, FLAME_E_INVAL, "lam is NULL");
  hipError_t e = by_storage(c, [&](auto tag) {
    using S = decltype(tag);
    using R = typename Enc<S>::R;
    hipLaunchKernelGGL(adjoint_fields_kernel<S>, dim3(blocks_for(c->n, 256)), dim3(256), 0, c->stream,
                       make_view<S>(c), static_cast<const R*>(c->p.force_u), dl_du, dl_db, static_cast<R*>(lam));
    return hipGetLastError();
  });
  if (e != hipSuccess) return fail(c, FLAME_E_HIP, std::string("field adjoint kernel: ") + hipGetErrorString(e));
  return FLAME_OK;
}

int64_t flame_step_count(const flame_ctx* c) { return c ? c->steps : -1; }

double flame_cfl_number(const flame_ctx* c) { return c ? c->cfl : 0.0; }

const char* flame_last_error(const flame_ctx* c) { return c ? c->err.c_str() : g_init_error.c_str(); }

void flame_destroy(flame_ctx* c) {
  if (!c) return;
  (void)hipStreamSynchronize(c->stream);
  if (c->plan_ok) hipfftDestroy(c->plan);
  if (c->plan_inv_ok) hipfftDestroy(c->plan_inv);
  if (c->red_partials) (void)hipFree(c->red_partials);
  if (c->fft_work) (void)hipFree(c->fft_work);
  if (c->spec_work) (void)hipFree(c->spec_work);
  if (c->transfer_work) (void)hipFree(c->transfer_work);
  if (c->spec_partials) (void)hipFree(c->spec_partials);
  delete c;
}

}  // extern "C"
