// Instantiations of the register-staged projection kernel, float32 (split into bf16 pieces), 64-row tiles.
#include "k1_stage.hpp"

namespace kb {
hipError_t launch_k1_stage_f32_L64(int kc, dim3 grid, const K1Args& a, hipStream_t st) {
  return launch_k1_stage<LayL64, true>(kc, grid, a, st);
}
hipError_t launch_k1_stage_f32_L64M(int kc, dim3 grid, const K1Args& a, hipStream_t st) {
  return launch_k1_stage<LayL64M, true>(kc, grid, a, st);
}
}  // namespace kb
