// Instantiations of the register-staged projection kernel, float32 (split into bf16 pieces), 32-row tiles of 256 and 128 words.
#include "k1_stage.hpp"

namespace kb {
hipError_t launch_k1_stage_f32_L32M(int kc, dim3 grid, const K1Args& a, hipStream_t st) {
  return launch_k1_stage<LayL32M, true>(kc, grid, a, st);
}
hipError_t launch_k1_stage_f32_L32S(int kc, dim3 grid, const K1Args& a, hipStream_t st) {
  return launch_k1_stage<LayL32S, true>(kc, grid, a, st);
}
}  // namespace kb
