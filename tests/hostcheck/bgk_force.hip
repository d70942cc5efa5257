// Host build of one node's BGK fluid collision in both arithmetic types (test infrastructure).
#include "../../paper_2212_11024_amd/csrc/flame_device.h"

using namespace flame;

template <typename R>
static void collide(const double* f_in, const double* b_in, const double* b0_in, const double* F_in, double omega,
                    double* f_out) {
  R f[kQ], F[3], b[3], b0[3];
  for (int i = 0; i < kQ; ++i) f[i] = R(f_in[i]);
  for (int c = 0; c < 3; ++c) {
    F[c] = R(F_in[c]);
    b[c] = R(b_in[c]);
    b0[c] = R(b0_in[c]);
  }
  const FluidMoments<R> m = fluid_moments(f);
  const R rho = R(1) + m.drho;
  const R U[3] = {(m.jx + R(0.5) * F[0]) / rho, (m.jy + R(0.5) * F[1]) / rho, (m.jz + R(0.5) * F[2]) / rho};
  collide_fluid_bgk(f, m, U, b, b0, F, R(omega));
  for (int i = 0; i < kQ; ++i) f_out[i] = double(f[i]);
}

extern "C" void bgk_collide(int single, const double* f, const double* b, const double* b0, const double* F, double omega,
                            double* out) {
  if (single) collide<float>(f, b, b0, F, omega, out);
  else collide<double>(f, b, b0, F, omega, out);
}
