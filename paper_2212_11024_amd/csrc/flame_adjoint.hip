// Adjoint of the time step (reverse mode): lam_t = (d step / d x_t)^T lam_{t+1}.
//
// A step is x_{t+1} = Stream(Collide(x_t)) with x the canonical (post-streaming) populations.
// Streaming moves population q from node y to y + c_q, so its transpose gathers: the adjoint of
// the post-collision population q at node y is lam_{t+1}[q] at y + c_q. The collision is
// node-local except, on the stencil route, through J = curl b, which couples a node to the field
// of its six face neighbours; that coupling is transposed in a second pass (the central-difference
// curl is its own transpose). Forward values are taken either from the state saved by the
// forward step (flame_step_save: the adjoint reads 51 values, gathers 48 and writes 48 per node)
// or, on the moment route, from a trace lattice (flame_adjoint_trace_step: the pre-collision
// state is pulled from the previous time level exactly as the forward step pulls it, and J is
// recomputed from it, so the recompute is one ordinary step and writes nothing extra).

#include "flame_access.h"
#include "flame_internal.h"

namespace flame {

template <typename R>
struct AdjArgs {
  const R* state;      // [48 + 3][n]: pre-collision deviations and J of the forward step
  const R* lam_next;   // [48][n]
  R* lam;              // [48][n]
  R* lam_j;            // [3][n] (stencil route)
  const R* force_u;
  const R* force_b;
  GridShape shape;
  size_t n;
  PhysConst<R> k;
};

// Bound by HBM: 100 loads and 48 stores per node. At least two waves per SIMD, which FP64 misses by a
// few registers otherwise (48^3 20.5 -> 19.2 us). The adjoints of the fluid populations are folded into
// 13 sums before the magnetic ones are needed, so neither kernel holds all 48 (FP32 115 registers).
// FP32 128^3 252 -> 223 us, 200^3 1238 -> 904; FP64 128^3 645 -> 442, 48^3 42 -> 19.
constexpr int kAdjThreads = 256;
// Addressing: 32-bit node offsets from the uniform array bases, by 64-bit global addresses (buffer
// resources run within 1% of them here). The entry points refuse arrays of more than 4 GiB.
//
// The adjoints of the next time level, gathered along the streaming: population q of node x went
// to x + c_q, so its adjoint is lam_next[q] there.
template <Addr A, typename R>
__device__ __forceinline__ void gather_next_fluid(const R* lam_next, size_t n, const Rows& rw, const Planes& pl,
                                                  R (&l)[kQ]) {
#pragma unroll
  for (int i = 0; i < kQ; ++i)
    l[tidx(cq(i, 0) + 1, cq(i, 1) + 1, cq(i, 2) + 1)] =
        ld<A>(lam_next + static_cast<size_t>(i) * n, rw.at(cq(i, 0), cq(i, 1)) + pl.at(cq(i, 2)));
}
template <Addr A, typename R>
__device__ __forceinline__ void gather_next_magnetic(const R* lam_next, size_t n, const Rows& rw, const Planes& pl,
                                                     R (&mg)[kM]) {
#pragma unroll
  for (int i = 0; i < 7; ++i) {
    const uint32_t dn = rw.at(xim(i, 0), xim(i, 1)) + pl.at(xim(i, 2));
#pragma unroll
    for (int c = 0; c < 3; ++c) mg[i * 3 + c] = ld<A>(lam_next + static_cast<size_t>(kQ + i * 3 + c) * n, dn);
  }
}

// The reverse pass of one node from its forward quantities: gathers the next adjoints, writes the
// node's (and, on the stencil route, lJ).
template <Addr A, typename R, bool MOMENT>
__device__ __forceinline__ void reverse_node(const VjpState<R>& fw, const R (&F)[3], const PhysConst<R>& k,
                                             const R* lam_next, R* lam, R* lam_j, size_t n, const Rows& rw,
                                             const Planes& pl, uint32_t cell) {
  NodeAdjoint<R> o;
  R l[kQ];
  gather_next_fluid<A>(lam_next, n, rw, pl, l);
  vjp_fluid(fw, F, k, l, o);
  R mg[kM], lJ[3];
  gather_next_magnetic<A>(lam_next, n, rw, pl, mg);
  vjp_magnetic<R, MOMENT>(fw, k, o, mg, lJ);
  vjp_fluid_populations(fw, o, l);
#pragma unroll
  for (int q = 0; q < kQ; ++q) st<A>(lam + static_cast<size_t>(q) * n, cell, l[q]);
#pragma unroll
  for (int q = 0; q < kM; ++q) st<A>(lam + static_cast<size_t>(kQ + q) * n, cell, mg[q]);
  if (!MOMENT) {
#pragma unroll
    for (int c = 0; c < 3; ++c) st<A>(lam_j + static_cast<size_t>(c) * n, cell, lJ[c]);
  }
}

template <typename R, bool MOMENT>
__global__ __launch_bounds__(kAdjThreads, 2) void adjoint_step_kernel(AdjArgs<R> a) {
  constexpr Addr A = Addr::Global;
  uint32_t cell;
  if (!own_cell(a.shape, cell)) return;
  const size_t n = a.n;
  const NodeAt at = NodeAt::of(cell, a.shape);
  const Rows& rw = at.rw;
  const Planes& pl = at.pl;
  R F[3];
  VjpState<R> fw;
  {
    R f[kQ], g[kM], J[3], S[3];
#pragma unroll
    for (int q = 0; q < kQ; ++q) f[q] = ld<A>(a.state + static_cast<size_t>(q) * n, cell);
#pragma unroll
    for (int q = 0; q < kM; ++q) g[q] = ld<A>(a.state + static_cast<size_t>(kQ + q) * n, cell);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      J[c] = ld<A>(a.state + static_cast<size_t>(kQ + kM + c) * n, cell);
      F[c] = a.force_u ? ld<A>(a.force_u + static_cast<size_t>(c) * n, cell) : R(0);
      S[c] = a.force_b ? ld<A>(a.force_b + static_cast<size_t>(c) * n, cell) : R(0);
    }
    fw = vjp_forward<R, MOMENT>(f, g, F, S, J, a.k);
  }
  reverse_node<A, R, MOMENT>(fw, F, a.k, a.lam_next, a.lam, a.lam_j, n, rw, pl, cell);
}

// Moment route from a trace lattice: the step's pre-collision state is the lattice pulled.
template <typename S>
struct AdjTraceArgs {
  using R = typename Enc<S>::R;
  const S* src;        // trace lattice [48][n] (storage encoding)
  const R* lam_next;   // [48][n]
  R* lam;              // [48][n]
  const R* force_u;
  const R* force_b;
  GridShape shape;
  size_t n;
  PhysConst<R> k;
};

template <typename S>
__global__ __launch_bounds__(kAdjThreads, 2) void adjoint_trace_kernel(AdjTraceArgs<S> a) {
  constexpr Addr A = Addr::Global;
  using E = Enc<S>;
  using R = typename E::R;
  uint32_t cell;
  if (!own_cell(a.shape, cell)) return;
  const size_t n = a.n;
  const NodeAt at = NodeAt::of(cell, a.shape);
  const Rows& rw = at.rw;
  const Planes& pl = at.pl;
  R F[3];
  VjpState<R> fw;
  {
    // the step's pre-collision state pulled from the lattice, and the forward step's J recomputed
    // from it (moment route, same order of operations)
    R f[kQ], g[kM], Sb[3];
#pragma unroll
    for (int i = 0; i < kQ; ++i)
      f[i] = E::dec(ld<A>(a.src + static_cast<size_t>(i) * n, rw.at(-cq(i, 0), -cq(i, 1)) + pl.at(-cq(i, 2))),
                    R(1.0 / E::fscale(i)));
#pragma unroll
    for (int i = 0; i < 7; ++i) {
      const uint32_t sn = rw.at(-xim(i, 0), -xim(i, 1)) + pl.at(-xim(i, 2));
#pragma unroll
      for (int c = 0; c < 3; ++c)
        g[i * 3 + c] = E::dec(ld<A>(a.src + static_cast<size_t>(kQ + i * 3 + c) * n, sn), R(1.0 / E::mscale(i)));
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      F[c] = a.force_u ? ld<A>(a.force_u + static_cast<size_t>(c) * n, cell) : R(0);
      Sb[c] = a.force_b ? ld<A>(a.force_b + static_cast<size_t>(c) * n, cell) : R(0);
    }
    const R unused[3] = {R(0), R(0), R(0)};
    fw = vjp_forward<R, true>(f, g, F, Sb, unused, a.k);
  }
  reverse_node<A, R, true>(fw, F, a.k, a.lam_next, a.lam, static_cast<R*>(nullptr), n, rw, pl, cell);
}

// Stencil route: b_c of every magnetic population set feeds J of the six face neighbours; add
// curl(lam_J) (the transpose of the central-difference curl) to the adjoint of all 7 g_{i,c}.
template <typename R>
__global__ __launch_bounds__(kAdjThreads) void adjoint_curl_kernel(R* lam, const R* lam_j, GridShape shape, size_t n) {
  constexpr Addr A = Addr::Global;
  uint32_t cell;
  if (!own_cell(shape, cell)) return;
  const NodeAt at = NodeAt::of(cell, shape);
  auto L = [&](int c, int dx, int dy, int dz) {
    return ld<A>(lam_j + static_cast<size_t>(c) * n, at.rw.at(dx, dy) + at.pl.at(dz));
  };
  const R cx = R(0.5) * (L(2, 0, 1, 0) - L(2, 0, -1, 0)) - R(0.5) * (L(1, 0, 0, 1) - L(1, 0, 0, -1));
  const R cy = R(0.5) * (L(0, 0, 0, 1) - L(0, 0, 0, -1)) - R(0.5) * (L(2, 1, 0, 0) - L(2, -1, 0, 0));
  const R cz = R(0.5) * (L(1, 1, 0, 0) - L(1, -1, 0, 0)) - R(0.5) * (L(0, 0, 1, 0) - L(0, 0, -1, 0));
  const R cc[3] = {cx, cy, cz};
#pragma unroll
  for (int i = 0; i < 7; ++i)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      R* base = lam + static_cast<size_t>(kQ + i * 3 + c) * n;
      st<A, false>(base, cell, ld<A>(base, cell) + cc[c]);
    }
}

// Adjoint of the initial state: d loss / d(u, b, grad u, grad b) from lam_0.
template <typename R>
struct InitAdjArgs {
  const R* lam0;
  const double* u;
  const double* b;
  const double* gu;
  const double* gb;
  const R* force_u;
  double* out_u;
  double* out_b;
  double* out_gu;
  double* out_gb;
  size_t n;
  PhysConst<double> k;
  InitFlags fl;
};

template <typename R>
__global__ __launch_bounds__(256) void init_vjp_kernel(InitAdjArgs<R> a) {
  const size_t cell = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (cell >= a.n) return;
  const size_t n = a.n;
  double u[3], b[3], G[3][3] = {}, H[3][3] = {}, F[3], lf[kQ], lg[kM];
  for (int c = 0; c < 3; ++c) {
    u[c] = a.u[c * n + cell];
    b[c] = a.b[c * n + cell];
    F[c] = a.force_u ? static_cast<double>(a.force_u[c * n + cell]) : 0.0;
  }
  if (a.gu)
    for (int p = 0; p < 3; ++p)
      for (int q = 0; q < 3; ++q) G[p][q] = a.gu[(p * 3 + q) * n + cell];
  if (a.gb)
    for (int p = 0; p < 3; ++p)
      for (int q = 0; q < 3; ++q) H[p][q] = a.gb[(p * 3 + q) * n + cell];
  for (int q = 0; q < kQ; ++q) lf[q] = static_cast<double>(a.lam0[q * n + cell]);
  for (int q = 0; q < kM; ++q) lg[q] = static_cast<double>(a.lam0[(kQ + q) * n + cell]);
  double ou[3], ob[3], oG[3][3], oH[3][3];
  init_node_vjp(u, b, G, H, F, a.k, a.fl, lf, lg, ou, ob, oG, oH);
  for (int c = 0; c < 3; ++c) {
    a.out_u[c * n + cell] = ou[c];
    a.out_b[c * n + cell] = ob[c];
  }
  if (a.out_gu)
    for (int p = 0; p < 3; ++p)
      for (int q = 0; q < 3; ++q) a.out_gu[(p * 3 + q) * n + cell] = oG[p][q];
  if (a.out_gb)
    for (int p = 0; p < 3; ++p)
      for (int q = 0; q < 3; ++q) a.out_gb[(p * 3 + q) * n + cell] = oH[p][q];
}

template <typename R>
static hipError_t adjoint_typed(const flame_ctx* c, const void* state, const void* lam_next, void* lam, void* lam_j) {
  AdjArgs<R> a;
  a.state = static_cast<const R*>(state);
  a.lam_next = static_cast<const R*>(lam_next);
  a.lam = static_cast<R*>(lam);
  a.lam_j = static_cast<R*>(lam_j);
  a.force_u = static_cast<const R*>(c->p.force_u);
  a.force_b = static_cast<const R*>(c->p.force_b);
  a.shape = grid_shape(c->p, row_threads(c->p.nx));
  a.n = c->n;
  a.k.omega = R(c->omega);
  a.k.omega_b = R(c->omega_b);
  a.k.alpha = R(c->p.d_i);
  for (int i = 0; i < 3; ++i) a.k.b0[i] = R(c->p.b0[i]);
  const dim3 grid(a.shape.blocks), block(a.shape.threads);
  if (c->p.jmode == FLAME_J_STENCIL) {
    hipLaunchKernelGGL((adjoint_step_kernel<R, false>), grid, block, 0, c->stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(adjoint_curl_kernel<R>, grid, block, 0, c->stream, a.lam, a.lam_j, a.shape, a.n);
  } else {
    hipLaunchKernelGGL((adjoint_step_kernel<R, true>), grid, block, 0, c->stream, a);
  }
  return hipGetLastError();
}

template <typename S>
static hipError_t adjoint_trace_typed(const flame_ctx* c, const void* src, const void* lam_next, void* lam) {
  using R = typename Enc<S>::R;
  AdjTraceArgs<S> a;
  a.src = static_cast<const S*>(src);
  a.lam_next = static_cast<const R*>(lam_next);
  a.lam = static_cast<R*>(lam);
  a.force_u = static_cast<const R*>(c->p.force_u);
  a.force_b = static_cast<const R*>(c->p.force_b);
  a.shape = grid_shape(c->p, row_threads(c->p.nx));
  a.n = c->n;
  a.k.omega = R(c->omega);
  a.k.omega_b = R(c->omega_b);
  a.k.alpha = R(c->p.d_i);
  for (int i = 0; i < 3; ++i) a.k.b0[i] = R(c->p.b0[i]);
  const dim3 grid(a.shape.blocks), block(a.shape.threads);
  hipLaunchKernelGGL(adjoint_trace_kernel<S>, grid, block, 0, c->stream, a);
  return hipGetLastError();
}

template <typename R>
static hipError_t init_vjp_typed(const flame_ctx* c, const void* lam0, const double* u, const double* b,
                                 const double* gu, const double* gb, double* ou, double* ob, double* ogu,
                                 double* ogb) {
  InitAdjArgs<R> a;
  a.lam0 = static_cast<const R*>(lam0);
  a.u = u;
  a.b = b;
  a.gu = gu;
  a.gb = gb;
  a.force_u = static_cast<const R*>(c->p.force_u);
  a.out_u = ou;
  a.out_b = ob;
  a.out_gu = ogu;
  a.out_gb = ogb;
  a.n = c->n;
  a.k.omega = c->omega;
  a.k.omega_b = c->omega_b;
  a.k.alpha = c->p.d_i;
  for (int i = 0; i < 3; ++i) a.k.b0[i] = c->p.b0[i];
  a.fl.fluid_noneq = c->p.init_noneq && gu;
  a.fl.mag_noneq = c->p.init_noneq && gb;
  a.fl.has_H = gb != nullptr;
  hipLaunchKernelGGL(init_vjp_kernel<R>, dim3((c->n + 255) / 256), dim3(256), 0, c->stream, a);
  return hipGetLastError();
}

// Every [n] array of the arithmetic type within 4 GiB (32-bit byte offsets in the kernels).
static bool adjoint_arrays_fit(flame_ctx* c) {
  const size_t bytes = c->n * (c->p.storage == FLAME_F64 ? 8 : 4);
  if (bytes <= (size_t(1) << 32)) return true;
  c->err = "reverse mode: each [n] array of the arithmetic type must fit in 4 GiB";
  return false;
}

}  // namespace flame

using namespace flame;

extern "C" {

flame_status flame_step_save(flame_ctx* c, void* state) {
  if (!c) return FLAME_E_INVAL;
  if (!reverse_mode_built(c->p)) {
    c->err = "reverse mode is built for the paper's model only (central-moment fluid, Hall equilibrium, "
             "D3Q27 / D3Q7 velocity sets)";
    return FLAME_E_UNSUPPORTED;
  }
  if (!state) {
    c->err = "state is NULL";
    return FLAME_E_INVAL;
  }
  if (!adjoint_arrays_fit(c)) return FLAME_E_INVAL;
  const SetPtrs ptr = set_ptrs(c);
  hipError_t e = launch_step(c, ptr, c->stride, state);
  if (e != hipSuccess) {
    c->err = std::string("step kernel: ") + hipGetErrorString(e);
    return FLAME_E_HIP;
  }
  const bool two_f = c->p.layout == FLAME_LAYOUT_AB;
  const bool two_g = mag_two_lattice(c->p);
  if (two_f || two_g) c->cur ^= 1;
  if (!two_f || !two_g) c->parity ^= 1;
  c->steps += 1;
  return FLAME_OK;
}

flame_status flame_trace_step(flame_ctx* c, const void* src, void* dst) {
  if (!c) return FLAME_E_INVAL;
  if (!reverse_mode_built(c->p)) {
    c->err = "reverse mode is built for the paper's model only (central-moment fluid, Hall equilibrium, "
             "D3Q27 / D3Q7 velocity sets)";
    return FLAME_E_UNSUPPORTED;
  }
  if (c->p.jmode != FLAME_J_MOMENT || c->p.layout != FLAME_LAYOUT_AA) {
    c->err = "trace step is available on the moment route with the AA layout only";
    return FLAME_E_UNSUPPORTED;
  }
  if (!src || !dst || src == dst) {
    c->err = "trace step needs distinct src and dst";
    return FLAME_E_INVAL;
  }
  const size_t set = 27 * c->n * value_bytes(c->p.storage);
  SetPtrs s{};
  s.f_src = const_cast<void*>(src);
  s.g_src = static_cast<char*>(s.f_src) + set;
  s.f_dst = dst;
  s.g_dst = static_cast<char*>(dst) + set;
  s.fluid_aa = false;
  s.mag_aa = false;
  hipError_t e = launch_step(c, s, c->n, nullptr);
  if (e != hipSuccess) {
    c->err = std::string("step kernel: ") + hipGetErrorString(e);
    return FLAME_E_HIP;
  }
  return FLAME_OK;
}

flame_status flame_adjoint_step(flame_ctx* c, const void* state, const void* lam_next, void* lam, void* lam_j) {
  if (!c) return FLAME_E_INVAL;
  if (!reverse_mode_built(c->p)) {
    c->err = "reverse mode is built for the paper's model only (central-moment fluid, Hall equilibrium, "
             "D3Q27 / D3Q7 velocity sets)";
    return FLAME_E_UNSUPPORTED;
  }
  if (!state || !lam_next || !lam || lam == lam_next || (c->p.jmode == FLAME_J_STENCIL && !lam_j)) {
    c->err = "adjoint step needs state, lam_next and a distinct lam (and lam_j for the stencil route)";
    return FLAME_E_INVAL;
  }
  if (!adjoint_arrays_fit(c)) return FLAME_E_INVAL;
  hipError_t e = c->p.storage == FLAME_F64 ? adjoint_typed<double>(c, state, lam_next, lam, lam_j)
                                           : adjoint_typed<float>(c, state, lam_next, lam, lam_j);
  if (e != hipSuccess) {
    c->err = std::string("adjoint kernel: ") + hipGetErrorString(e);
    return FLAME_E_HIP;
  }
  return FLAME_OK;
}

flame_status flame_adjoint_trace_step(flame_ctx* c, const void* src, const void* lam_next, void* lam) {
  if (!c) return FLAME_E_INVAL;
  if (!reverse_mode_built(c->p)) {
    c->err = "reverse mode is built for the paper's model only (central-moment fluid, Hall equilibrium, "
             "D3Q27 / D3Q7 velocity sets)";
    return FLAME_E_UNSUPPORTED;
  }
  if (c->p.jmode != FLAME_J_MOMENT || c->p.layout != FLAME_LAYOUT_AA) {
    c->err = "the trace adjoint is available on the moment route with the AA layout only";
    return FLAME_E_UNSUPPORTED;
  }
  if (!src || !lam_next || !lam || lam == lam_next) {
    c->err = "trace adjoint needs src, lam_next and a distinct lam";
    return FLAME_E_INVAL;
  }
  if (!adjoint_arrays_fit(c)) return FLAME_E_INVAL;
  hipError_t e;
  switch (c->p.storage) {
    case FLAME_F64: e = adjoint_trace_typed<double>(c, src, lam_next, lam); break;
    case FLAME_F32: e = adjoint_trace_typed<float>(c, src, lam_next, lam); break;
    default: e = adjoint_trace_typed<_Float16>(c, src, lam_next, lam); break;
  }
  if (e != hipSuccess) {
    c->err = std::string("adjoint kernel: ") + hipGetErrorString(e);
    return FLAME_E_HIP;
  }
  return FLAME_OK;
}

flame_status flame_adjoint_init(flame_ctx* c, const void* lam0, const double* u, const double* b,
                                const double* grad_u, const double* grad_b, double* g_u, double* g_b,
                                double* g_grad_u, double* g_grad_b) {
  if (!c) return FLAME_E_INVAL;
  if (!reverse_mode_built(c->p)) {
    c->err = "reverse mode is built for the paper's model only (central-moment fluid, Hall equilibrium, "
             "D3Q27 / D3Q7 velocity sets)";
    return FLAME_E_UNSUPPORTED;
  }
  if (!lam0 || !u || !b || !g_u || !g_b) {
    c->err = "adjoint init needs lam0, u, b, g_u and g_b";
    return FLAME_E_INVAL;
  }
  if (c->p.init_noneq && (!grad_u || !grad_b)) {
    c->err = "adjoint init needs the gradients that flame_init received (the transpose of the "
             "central differences taken in their absence is not built)";
    return FLAME_E_UNSUPPORTED;
  }
  hipError_t e = c->p.storage == FLAME_F64
                     ? init_vjp_typed<double>(c, lam0, u, b, grad_u, grad_b, g_u, g_b, g_grad_u, g_grad_b)
                     : init_vjp_typed<float>(c, lam0, u, b, grad_u, grad_b, g_u, g_b, g_grad_u, g_grad_b);
  if (e != hipSuccess) {
    c->err = std::string("initial-state adjoint kernel: ") + hipGetErrorString(e);
    return FLAME_E_HIP;
  }
  return FLAME_OK;
}

}  // extern "C"
