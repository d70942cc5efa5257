// Host-side context and launcher declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <hipfft/hipfft.h>

#include <algorithm>
#include <string>

#include "../../include/flame.h"
#include "flame_device.h"

struct flame_ctx {
  flame_params p{};
  int device = 0;
  int cus = 0;               // compute units of the device
  hipStream_t stream = nullptr;
  size_t n = 0;              // nodes
  size_t stride = 0;         // elements between consecutive population arrays
  void* storage = nullptr;   // caller-owned populations
  int parity = 0;            // AA in-place sets: 0 = canonical slots, 1 = swapped slots
  int cur = 0;               // two-lattice sets: index of the copy holding the current state
  int64_t steps = 0;
  double frest[27]{};        // f^mhd(0)(1, 0, b0)
  double omega = 0, omega_b = 0;
  double cfl = 0;
  // launch shape (tuning; read from the environment at flame_init, results do not depend on it):
  // planes per workgroup of the stencil kernel (0: by the grid's size) and threads per row block of
  // the node-local kernels (0: the row rounded up to whole wavefronts, at most 256)
  int zchunk = 0;
  int row_tx = 0;
  bool global_addr = false;   // FLAME_GLOBAL_ADDRESSING=1: no buffer addressing in the step
  std::string err;
  // library-owned scratch
  double* red_partials = nullptr;
  int red_blocks = 0;
  double* scratch = nullptr;   // this device's static reduction scratch (not owned)
  hipfftDoubleComplex* spec_work = nullptr;   // spec_batch components, transformed in place
  size_t spec_work_size = 0;
  int spec_batch = 0;                         // components per transform: 3 or 1 (0: not decided yet)
  double* spec_partials = nullptr;            // block partials and merged rows of the shell sums
  size_t spec_partials_size = 0;
  hipfftDoubleComplex* transfer_work = nullptr;   // fields and transforms of the energy transfer
  size_t transfer_size = 0;
  char* fft_work = nullptr;                   // work area of both plans, which run one after the other
  size_t fft_work_size = 0;
  size_t plan_work = 0, plan_inv_work = 0;    // bytes of it that each plan needs
  hipfftHandle plan{};
  bool plan_ok = false;
  hipfftHandle plan_inv{};   // complex-to-real inverse, for spectral derivatives
  bool plan_inv_ok = false;
};

namespace flame {

// Pointers to the population sets of the current step.
struct SetPtrs {
  void* f_src;
  void* f_dst;
  void* g_src;
  void* g_dst;
  bool fluid_aa;     // fluid set updated in place (else two-lattice pull)
  bool mag_aa;       // magnetic set updated in place (else two-lattice pull)
};

inline size_t value_bytes(int storage) { return storage == FLAME_F64 ? 8 : storage == FLAME_F32 ? 4 : 2; }

// Population arrays are laid out back to back with a stride of the node count rounded up to
// 256 bytes plus a pad, so that the 48 arrays do not all start at large powers of two apart.
#ifndef FLAME_STRIDE_PAD_BYTES
#define FLAME_STRIDE_PAD_BYTES 0
#endif
inline size_t population_stride(const flame_params& p) {
  const size_t vb = value_bytes(p.storage);
  const size_t n = static_cast<size_t>(p.nx) * p.ny * p.nz;
  const size_t align = 256 / vb;
  return (n + align - 1) / align * align + FLAME_STRIDE_PAD_BYTES / vb;
}
// The node-local step may address its arrays through buffer resources (32-bit offsets, range
// limit 2^32 - 1 bytes) only when every array it touches ends at least 16 bytes below 4 GiB, so
// that no access can meet the range limit whichever byte of it the hardware checks: the
// population arrays, and, when the launch reads forcing or writes a saved state
// (arith_arrays), the [n] arrays of the arithmetic type. Larger arrays take the 64-bit global
// addresses instead.
inline bool buffer_addressing_ok(const flame_params& p, bool arith_arrays) {
  const size_t limit = (size_t(1) << 32) - 16;
  const size_t n = static_cast<size_t>(p.nx) * p.ny * p.nz;
  const size_t arith = p.storage == FLAME_F64 ? 8 : 4;
  return population_stride(p) * value_bytes(p.storage) <= limit && (!arith_arrays || n * arith <= limit);
}
// Model bits of the step kernels: 1 = BGK fluid collision, 2 = electron MHD; 0 is the paper's.
inline int step_model(const flame_params& p) {
  return (p.collision == FLAME_COLLISION_BGK ? 1 : 0) | (p.magnetic == FLAME_MAGNETIC_EMHD ? 2 : 0);
}
inline bool mag_two_lattice(const flame_params& p) {
  return p.layout == FLAME_LAYOUT_AB || p.jmode == FLAME_J_STENCIL;
}
// Velocity sets: a run on anything but the paper's D3Q27 fluid and D3Q7 magnetic sets goes
// through the lattice-variant kernels (flame_lattice.hip).
inline bool lattice_variant(const flame_params& p) {
  return p.fluid_lattice != FLAME_FLUID_D3Q27 || p.magnetic_lattice != FLAME_MAGNETIC_D3Q7;
}
inline int fluid_count(const flame_params& p) { return p.fluid_lattice == FLAME_FLUID_D3Q19 ? 19 : 27; }
inline int mag_count(const flame_params& p) {
  return p.magnetic_lattice == FLAME_MAGNETIC_D3Q15 ? 15 : p.magnetic_lattice == FLAME_MAGNETIC_D3Q27 ? 27 : 7;
}
// Reverse mode and trace lattices are built for the paper's model and velocity sets only.
inline bool reverse_mode_built(const flame_params& p) { return step_model(p) == 0 && !lattice_variant(p); }
SetPtrs set_ptrs(const flame_ctx* c);

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own L2): hardware
// workgroup h runs on XCD h % 8. Remap so that XCD j processes one contiguous range of logical
// tiles (x fastest, then y, then z): neighbouring tiles, which share halo rows and the cache
// lines that shifted stores straddle, then sit behind the same L2.
#ifndef FLAME_XCD_REMAP
#define FLAME_XCD_REMAP 1
#endif
constexpr unsigned kXCDs = 8;

__device__ __forceinline__ unsigned logical_index(unsigned total) {
  const unsigned h = blockIdx.x;
  if (!FLAME_XCD_REMAP) return h;
  const unsigned q = total / kXCDs, r = total % kXCDs;
  const unsigned j = h % kXCDs, k = h / kXCDs;
  return j * q + min(j, r) + k;
}
__device__ __forceinline__ void logical_block(unsigned gx, unsigned gy, unsigned gz, unsigned& bx, unsigned& by,
                                              unsigned& bz) {
  const unsigned l = logical_index(gx * gy * gz);
  bx = l % gx;
  by = (l / gx) % gy;
  bz = l / (gx * gy);
}

// Grid extents of the kernels that split the grid by linear node index, with floor(2^32 / d) for
// the divisions by a row and by a plane. flame_init refuses grids of 2^32 nodes or more.
struct Divisor {
  uint32_t d, inv;
};
struct GridShape {
  Divisor nx, plane;
  uint32_t n;
  uint32_t threads, blocks;   // launch shape, as an argument: blockDim is a load that every address waits for
};
inline Divisor divisor(uint32_t d) { return {d, static_cast<uint32_t>(std::min<uint64_t>((uint64_t(1) << 32) / d, UINT32_MAX))}; }
inline GridShape grid_shape(const flame_params& p, unsigned threads) {
  const size_t n = static_cast<size_t>(p.nx) * p.ny * p.nz;
  return {divisor(static_cast<uint32_t>(p.nx)), divisor(static_cast<uint32_t>(p.nx) * p.ny), static_cast<uint32_t>(n),
          threads, static_cast<uint32_t>((n + threads - 1) / threads)};
}

// Planes per workgroup of a kernel that marches tiles along z: the power of two up to most that a grid
// finishes first with, counting rounds of resident workgroups times the planes of one, whose prologue
// costs about 3/4 of a plane. Long chunks waste less in prologues, short ones fill the chip.
inline int march_planes(int64_t tiles, int nz, int64_t resident, int most) {
  resident = std::max<int64_t>(resident, 1);
  int best = 1;
  double least = 0;
  for (int planes = 1; planes <= most; planes *= 2) {
    const int64_t groups = tiles * ((nz + planes - 1) / planes);
    const double cost = static_cast<double>((groups + resident - 1) / resident) * (std::min(planes, nz) + 0.75);
    if (planes == 1 || cost <= least) {
      least = cost;
      best = planes;
    }
  }
  return best;
}

// Whether the node-local step stores the lattice with the non-temporal hint; state: bytes of one lattice.
//
// Between two lattices: where both together are far beyond the 256 MB last-level cache, so that nothing
// written is read from it again (161 x 130 x 99 FP32 156 against 161 us a step, 100^3 FP64 149 against 153);
// below, the next step finds the lattice there (64^3 FP32 18.5 against 23.5 us, 48^3 FP64 16 against 20.5).
//
// In place: plain, because plain lines stay in L2 until the neighbouring wavefronts have filled those that
// shifted stores share (two steps, plain against hinted: FP32 64^3 33 against 40.5 us, 112^3 188 against 203,
// 132^3 372 against 386, 160^3 657 against 708, 200^3 1250 against 1337; FP64 88^3 161 against 182, 112^3 446
// against 455, 200^3 2460 against 2615; FP16 160^3 342 against 350). Except for FP32 and FP64 states a
// little larger than the cache, of which the hint leaves the part that is read next (FP32 122^3 282 against
// 265, 128^3 316 against 310, 161 x 130 x 99 322 against 318, 64 x 64 x 512 319 against 314; FP64 96^3 250
// against 235, 100^3 300 against 272, 104^3 353 against 346). The ends: FP32 118^3 (301 MiB) 235 against 245
// and 130^3 (402 MiB) 349 against 358, FP64 94^3 (304 MiB) 226 against 228 and 106^3 (436 MiB) as fast either way.
//
// Steps that also save their state write about as much again, 51 arrays that are not read soon, always with the
// hint. Their lattice follows the same rule in place, with the hint up to larger FP64 states (two steps, plain
// against hinted: FP32 96^3 157 against 217 us, 160^3 1037 against 1070, 200^3 1920 against 2034, 128^3 494 against
// 481; FP64 64^3 97 against 108, 92^3 340 against 322, 108^3 598 against 540, 112^3 670 against 616, 120^3 823
// against 822, 128^3 955 against 968, 200^3 3818 against 3958; FP16 96^3 112 against 143), and keeps it
// between two lattices (FP32 256^3 3935 against 4012 us, 96^3 222 against 237).
constexpr size_t kMiB = size_t(1) << 20;
inline bool nt_stores(bool two_lattices, bool save, size_t value_bytes, size_t state) {
  if (two_lattices) return save || 2 * state > 384 * kMiB;
  return value_bytes > 2 && state > 310 * kMiB && state <= (value_bytes == 4 ? 396 : save ? 640 : 416) * kMiB;
}

// LDS reserved by a block of the node-local step, so that fewer blocks share a compute unit and fewer rows
// in flight keep the lines that shifted accesses share in L2. FP32 states from 6 GiB on (2^25 nodes): three
// blocks of 256 threads instead of four to six (two steps, without and with: 336^3 6.07 and 5.92 ms, 384^3 8.88 and
// 8.70, 448^3 14.3 and 13.9, 512^3 20.3 and 20.0; trace steps 512^3 16.76 and 16.70; at 256^3 2.67 and 2.75, at 288^3 3.76
// and 3.69, 320^3 5.18 and 5.07, where the rule forgoes 2%). State-saving FP32 and FP16 steps, which
// write 99 arrays, from 264 MiB on: two blocks (160^3 FP32 1037 and 976 us, 256^3 4.20 and 3.90 ms, 512^3 in place
// 28.5 and 28.0; FP16 144^3 546 and 507 us, 256^3 2.96 and 2.59 ms; between two lattices FP32 256^3 3.94 and 3.84 ms,
// FP16 192^3 1185 and 1114 us; below, FP32 112^3 269 and 278 us, FP16 128^3 246 and 283), but not in place with the
// hint (FP32 128^3 481 and 497 us). FP64's registers bound its blocks.
constexpr unsigned kThreeBlocksLds = 50000, kTwoBlocksLds = 78000;   // of the 160 KB of a compute unit
inline unsigned reserved_lds(bool two_lattices, bool save, size_t value_bytes, size_t state) {
  if (save)
    return value_bytes < 8 && state > 264 * kMiB && (two_lattices || !nt_stores(false, true, value_bytes, state))
               ? kTwoBlocksLds : 0;
  return value_bytes == 4 && state >= 6144 * kMiB ? kThreeBlocksLds : 0;
}

// Whether the curl-stencil step runs one workgroup on a compute unit where its registers allow two (the even
// and two-lattice steps in FP32 and FP16). Two are a loss in FP32 unless forcing is read, which leaves
// more to wait for (two steps, two workgroups against one: 200^3 1749 against 1678 us, 240^3 2585 against 2400,
// 256^3 3020 against 2975 and between two lattices 2820 against 2625, 352^3 7750 against 7240, 384^3 9745
// against 9390, 512^3 23.3 against 22.6 ms; 160^3 709 against 714 us). Forced FP32 steps keep two (even
// step 160^3 355 against 404 us, 320^3 2735 against 2780), as do those of FP16 (256^3 1666 against 1696).
inline bool one_group_per_cu(const flame_params& p) { return p.storage == FLAME_F32 && !p.force_u && !p.force_b; }

// Threads per block of the node-local kernels: a row of nx nodes rounded up to whole wavefronts, at
// most 256 (their launch bound), whatever FLAME_ROW_THREADS asks for. The blocks of the kernels that
// split the grid by linear node index need not hold whole rows; there short rows only make blocks
// small, which spreads a small grid over more compute units.
constexpr int kRowThreadsMax = 256;
inline unsigned row_threads(int nx) { return static_cast<unsigned>(std::min(kRowThreadsMax, (nx + 63) / 64 * 64)); }
inline unsigned row_threads(const flame_ctx* c) {
  return c->row_tx > 0 ? static_cast<unsigned>(std::min({c->row_tx, kRowThreadsMax, (c->p.nx + 63) / 64 * 64}))
                       : row_threads(c->p.nx);
}

// One fused step over the sets s, whose population arrays are stride elements apart; with
// save != null also writes the pre-collision state of every node (arithmetic type,
// [48 populations + 3 J][n]).
hipError_t launch_step(const flame_ctx* c, const SetPtrs& s, size_t stride, void* save);

// Lattice-variant kernels (flame_lattice.hip), each enqueued on the context's stream.
hipError_t variant_launch_step(const flame_ctx* c, const SetPtrs& s);
hipError_t variant_launch_init(const flame_ctx* c, const double* u, const double* b, const double* grad_u,
                               const double* grad_b);
hipError_t variant_launch_get(const flame_ctx* c, int deviations, double* dst);
hipError_t variant_launch_gather(const flame_ctx* c, int deviations, const int64_t* cells, int64_t cnt, double* out);
hipError_t variant_launch_set(const flame_ctx* c, int deviations, const double* src);
hipError_t variant_launch_moments(const flame_ctx* c, double* rho, double* u, double* b, double* j, double* divb);
hipError_t variant_launch_components(const flame_ctx* c, int field, int first, int count, uint32_t pitch, size_t dist,
                                     double* out);
hipError_t variant_launch_reduce(const flame_ctx* c, double* partials);
// Rest populations of the lattice variants (host): f_rest[q], g_rest[3 m].
void variant_rest(const flame_params& p, double* f_rest, double* g_rest);

}  // namespace flame
