// Host build of the index arithmetic of the kernels that split the grid by linear node index, and
// of the plane count of the marching kernels (test infrastructure).
#include "../../paper_2212_11024_amd/csrc/flame_access.h"

using namespace flame;

extern "C" {

uint32_t nb_divide(uint32_t t, uint32_t d, uint32_t* rest) { return div_by(t, divisor(d), *rest); }

// The 27 neighbour indices of a node, order ((dz * 3) + dy) * 3 + dx, each offset by one.
void nb_neighbours(int nx, int ny, int nz, uint32_t cell, uint32_t* out) {
  flame_params p{};
  p.nx = nx;
  p.ny = ny;
  p.nz = nz;
  const NodeAt at = NodeAt::of(cell, grid_shape(p, 256));
  for (int z = -1; z <= 1; ++z)
    for (int y = -1; y <= 1; ++y)
      for (int x = -1; x <= 1; ++x) out[((z + 1) * 3 + y + 1) * 3 + x + 1] = at.rw.at(x, y) + at.pl.at(z);
}

int nb_march_planes(int64_t tiles, int nz, int64_t resident, int most) { return march_planes(tiles, nz, resident, most); }

}  // extern "C"
