// Host build of the rules by which launches are shaped (test infrastructure).
#include "../../paper_2212_11024_amd/csrc/flame_internal.h"

extern "C" {

int lr_one_group_per_cu(int storage, int forced) {
  flame_params p{};
  p.storage = storage;
  p.force_b = forced ? &p : nullptr;
  return flame::one_group_per_cu(p);
}

}  // extern "C"

static size_t state(int value_bytes, int nx, int ny, int nz) { return size_t(48) * value_bytes * nx * ny * nz; }
extern "C" int lr_nt_stores(int two_lattices, int save, int value_bytes, int nx, int ny, int nz) {
  return flame::nt_stores(two_lattices != 0, save != 0, value_bytes, state(value_bytes, nx, ny, nz));
}
extern "C" unsigned lr_reserved_lds(int two_lattices, int save, int value_bytes, int nx, int ny, int nz) {
  return flame::reserved_lds(two_lattices != 0, save != 0, value_bytes, state(value_bytes, nx, ny, nz));
}
