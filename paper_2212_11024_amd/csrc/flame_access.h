// Array access of the step and adjoint kernels: 32-bit node offsets from wave-uniform array
// bases, by 64-bit global addresses or by buffer resources.
#ifndef FLAME_ACCESS_H
#define FLAME_ACCESS_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "flame_device.h"
#include "flame_internal.h"

namespace flame {

#ifndef FLAME_NT_STORES
#define FLAME_NT_STORES 1
#endif

// Addresses: every array is indexed from a wave-uniform base (set + q * n, held in scalar
// registers) by a 32-bit per-lane node offset. A thread's nine in-plane neighbour offsets
// (x + dx, y + dy) are loop invariants; the plane offset z * nx * ny is uniform. The library
// limits each array to 4 GiB so byte offsets fit in 32 bits.
struct Rows {
  uint32_t r[3][3];   // [dx + 1][dy + 1] -> wrap(y + dy) * nx + wrap(x + dx)
  __device__ __forceinline__ Rows(int x, int y, int nx, int ny) {
#pragma unroll
    for (int dx = -1; dx <= 1; ++dx)
#pragma unroll
      for (int dy = -1; dy <= 1; ++dy)
        r[dx + 1][dy + 1] = static_cast<uint32_t>(wrap(y + dy, ny)) * nx + static_cast<uint32_t>(wrap(x + dx, nx));
  }
  // from x and the three row offsets y' * nx
  FLAME_HD Rows(uint32_t x, uint32_t nx, uint32_t below, uint32_t row, uint32_t above) {
    const uint32_t xs[3] = {x == 0 ? nx - 1 : x - 1, x, x + 1 == nx ? 0 : x + 1};
    const uint32_t ys[3] = {below, row, above};
#pragma unroll
    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
      for (int dy = 0; dy < 3; ++dy) r[dx][dy] = ys[dy] + xs[dx];
  }
  FLAME_HD uint32_t at(int dx, int dy) const { return r[dx + 1][dy + 1]; }
};

// Addressing of the arrays. Every array spans at most 4 GiB (checked by the entry points), so an
// access is a wave-uniform array base plus a 32-bit per-lane byte offset. Global:
// 64-bit flat-global addresses formed per access in vector registers. Buffer: a buffer resource
// per array (base in scalar registers, no range limit below 4 GiB, raw addressing) and the 32-bit
// offset as the only per-lane operand, which takes the 64-bit address arithmetic off the vector
// ALU (about 170 of the FP64 in-place odd step's 880 vector instructions per node).
enum class Addr { Global, Buffer };
typedef unsigned int U32x2 __attribute__((ext_vector_type(2)));
template <typename S>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const S* base) {
  // stride 0, num_records 2^32 - 1, dword 3 of a raw 32-bit-format buffer on gfx9
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<S*>(base), 0, 0xFFFFFFFF, 0x00020000);
}
template <Addr A, typename S>
__device__ __forceinline__ S ld(const S* base, uint32_t off) {
  const uint32_t vo = off * static_cast<uint32_t>(sizeof(S));
  if constexpr (A == Addr::Buffer) {
    if constexpr (sizeof(S) == 2)
      return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b16(rsrc_of(base), vo, 0, 0));
    else if constexpr (sizeof(S) == 4)
      return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(rsrc_of(base), vo, 0, 0));
    else
      return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(rsrc_of(base), vo, 0, 0));
  } else {
    return *reinterpret_cast<const S*>(reinterpret_cast<const char*>(base) + vo);
  }
}
// NT: with the non-temporal hint (unless FLAME_NT_STORES is 0).
template <Addr A, bool NT = true, typename S>
__device__ __forceinline__ void st(S* base, uint32_t off, S v) {
  constexpr bool nt = NT && FLAME_NT_STORES;
  const uint32_t vo = off * static_cast<uint32_t>(sizeof(S));
  if constexpr (A == Addr::Buffer) {
    constexpr int aux = nt ? 2 : 0;   // 2: the non-temporal hint
    if constexpr (sizeof(S) == 2)
      __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(short, v), rsrc_of(base), vo, 0, aux);
    else if constexpr (sizeof(S) == 4)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), rsrc_of(base), vo, 0, aux);
    else
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U32x2, v), rsrc_of(base), vo, 0, aux);
  } else {
    S* p = reinterpret_cast<S*>(reinterpret_cast<char*>(base) + vo);
    if (nt)
      __builtin_nontemporal_store(v, p);
    else
      *p = v;
  }
}

// Plane offsets of z - 1, z, z + 1 (periodic).
struct Planes {
  uint32_t p[3];
  FLAME_HD Planes(uint32_t below, uint32_t here, uint32_t above) : p{below, here, above} {}
  __device__ __forceinline__ Planes(int z, int nz, uint32_t plane) {
    p[0] = static_cast<uint32_t>(wrap(z - 1, nz)) * plane;
    p[1] = static_cast<uint32_t>(z) * plane;
    p[2] = static_cast<uint32_t>(wrap(z + 1, nz)) * plane;
  }
  FLAME_HD uint32_t at(int dz) const { return p[dz + 1]; }
};

// The node-local kernels split the grid by linear node index: a block owns g.threads consecutive
// nodes, whatever the row length, so every lane of every wavefront but the grid's last has a node
// and a block's own accesses start on a whole cache line also where the rows do not (a row per
// block leaves 16% of the lanes idle at nx = 161 and straddles a line at both ends of every wavefront).
// The division by nx and by the plane is a multiplication by floor(2^32 / d), one short at most.
FLAME_HD uint32_t div_by(uint32_t t, Divisor d, uint32_t& rest) {
  uint32_t q = static_cast<uint32_t>((static_cast<uint64_t>(t) * d.inv) >> 32);
  rest = t - q * d.d;
  if (rest >= d.d) {
    ++q;
    rest -= d.d;
  }
  return q;
}
struct NodeAt {
  uint32_t cell;
  Rows rw;
  Planes pl;
  static FLAME_HD NodeAt of(uint32_t cell, const GridShape& g) {
    uint32_t rem, x;
    const uint32_t z = div_by(cell, g.plane, rem);
    const uint32_t y = div_by(rem, g.nx, x);
    const uint32_t row = rem - x, here = cell - rem, nx = g.nx.d, plane = g.plane.d;
    return {cell,
            Rows(x, nx, y == 0 ? plane - nx : row - nx, row, row + nx == plane ? 0 : row + nx),
            Planes(z == 0 ? g.n - plane : here - plane, here, here + plane == g.n ? 0 : here + plane)};
  }
};
// The node of this thread, or false beyond the grid's end.
__device__ __forceinline__ bool own_cell(const GridShape& g, uint32_t& cell) {
  cell = logical_index(g.blocks) * g.threads + threadIdx.x;
  return cell < g.n;
}

}  // namespace flame

#endif
