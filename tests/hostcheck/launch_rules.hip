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
