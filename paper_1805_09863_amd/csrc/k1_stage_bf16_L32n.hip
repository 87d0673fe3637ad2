// Instantiations of the register-staged projection kernel, bf16, 32-row tiles of 256 and 128 words.
#include "k1_stage.hpp"

namespace kb {
hipError_t launch_k1_stage_bf16_L32M(int kc, dim3 grid, const K1Args& a, hipStream_t st) {
  return launch_k1_stage<LayL32M, false>(kc, grid, a, st);
}
hipError_t launch_k1_stage_bf16_L32S(int kc, dim3 grid, const K1Args& a, hipStream_t st) {
  return launch_k1_stage<LayL32S, false>(kc, grid, a, st);
}
}  // namespace kb
