// Host build of the library's spectral set-up over a device of limited memory (test infrastructure): the
// allocations and transform plans are replaced by counters, and nothing is launched.
#include <hip/hip_runtime.h>
#include <hipfft/hipfft.h>

#include <map>

namespace fake {
size_t room = 0;                 // bytes left
std::map<void*, size_t> held;    // allocations
std::map<size_t, size_t> plans;  // plan -> bytes of its own work area
size_t next = 1;
int fail_stream = 0, bad_release = 0;
double work_factor = 0;          // work area of a plan as a multiple of its half spectra
hipError_t alloc(void** p, size_t bytes) {
  if (bytes > room) return hipErrorOutOfMemory;
  room -= bytes;
  *p = reinterpret_cast<void*>(next++ << 12);
  held[*p] = bytes;
  return hipSuccess;
}
template <typename T>
hipError_t alloc(T** p, size_t bytes) { return alloc(reinterpret_cast<void**>(p), bytes); }
hipError_t release(void* p) {
  if (!held.count(p)) ++bad_release;
  else room += held[p];
  held.erase(p);
  return hipSuccess;
}
bool automatic = true;
hipfftResult create(hipfftHandle* h) {
  *h = reinterpret_cast<hipfftHandle>(next);
  plans[next++] = 0;
  automatic = true;
  return HIPFFT_SUCCESS;
}
hipfftResult set_auto(hipfftHandle, int on) {
  automatic = on != 0;
  return HIPFFT_SUCCESS;
}
hipfftResult make_many(hipfftHandle h, int, int* n, int*, int, int, int*, int, int, hipfftType, int batch, size_t* work) {
  *work = static_cast<size_t>(work_factor * 16.0 * batch * n[0] * n[1] * (n[2] / 2 + 1));
  if (!automatic) return HIPFFT_SUCCESS;
  if (*work > room) return HIPFFT_ALLOC_FAILED;
  room -= *work;
  plans[reinterpret_cast<size_t>(h)] = *work;
  return HIPFFT_SUCCESS;
}
hipfftResult set_stream(hipfftHandle, hipStream_t) { return fail_stream-- > 0 ? HIPFFT_INTERNAL_ERROR : HIPFFT_SUCCESS; }
hipfftResult set_area(hipfftHandle, void* p) { return held.count(p) ? HIPFFT_SUCCESS : HIPFFT_INVALID_VALUE; }
hipfftResult destroy(hipfftHandle h) {
  const size_t k = reinterpret_cast<size_t>(h);
  if (!plans.count(k)) ++bad_release;
  else room += plans[k];
  plans.erase(k);
  return HIPFFT_SUCCESS;
}
}  // namespace fake
#define hipMalloc(p, b) fake::alloc(p, b)
#define hipFree(p) fake::release(p)
#define hipGetLastError() hipSuccess
#define hipfftCreate(h) fake::create(h)
#define hipfftSetAutoAllocation(h, on) fake::set_auto(h, on)
#define hipfftMakePlanMany fake::make_many
#define hipfftSetStream(h, s) fake::set_stream(h, s)
#define hipfftSetWorkArea(h, p) fake::set_area(h, p)
#define hipfftDestroy(h) fake::destroy(h)

#include "../../paper_2212_11024_amd/csrc/flame_api.hip"

// No kernel is registered and none of the other translation units is reached.
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
}
namespace flame {
hipError_t launch_step(const flame_ctx*, const SetPtrs&, size_t, void*) { return hipErrorUnknown; }
void variant_rest(const flame_params&, double*, double*) {}
hipError_t variant_launch_get(const flame_ctx*, int, double*) { return hipErrorUnknown; }
hipError_t variant_launch_set(const flame_ctx*, int, const double*) { return hipErrorUnknown; }
hipError_t variant_launch_init(const flame_ctx*, const double*, const double*, const double*, const double*) {
  return hipErrorUnknown;
}
hipError_t variant_launch_gather(const flame_ctx*, int, const int64_t*, int64_t, double*) { return hipErrorUnknown; }
hipError_t variant_launch_reduce(const flame_ctx*, double*) { return hipErrorUnknown; }
hipError_t variant_launch_moments(const flame_ctx*, double*, double*, double*, double*, double*) { return hipErrorUnknown; }
hipError_t variant_launch_components(const flame_ctx*, int, int, int, uint32_t, size_t, double*) { return hipErrorUnknown; }
}  // namespace flame

extern "C" {

flame_ctx* ss_new(int nx, int ny, int nz, size_t room, double work_factor) {
  fake::room = room;
  fake::work_factor = work_factor;
  fake::fail_stream = fake::bad_release = 0;
  fake::held.clear();
  fake::plans.clear();
  flame_ctx* c = new flame_ctx;
  c->p.nx = nx;
  c->p.ny = ny;
  c->p.nz = nz;
  c->n = static_cast<size_t>(nx) * ny * nz;
  return c;
}
void ss_room(size_t room) { fake::room = room; }
void ss_fail_streams(int count) { fake::fail_stream = count; }
// transfer: bytes of the energy transfer's workspace (0: a spectrum)
int ss_setup(flame_ctx* c, int nshells, size_t transfer) {
  const int blocks = bin_blocks(half_shape(c), nshells);
  return spectral_setup(c, blocks, transfer ? 4 : 1, nshells, transfer != 0, transfer / sizeof(hipfftDoubleComplex));
}
int ss_batch(const flame_ctx* c) { return c->spec_batch; }
size_t ss_held() {
  size_t sum = 0;
  for (const auto& h : fake::held) sum += h.second;
  for (const auto& p : fake::plans) sum += p.second;
  return sum;
}
int ss_plans() { return static_cast<int>(fake::plans.size()); }
int ss_bad_releases() { return fake::bad_release; }

}  // extern "C"
