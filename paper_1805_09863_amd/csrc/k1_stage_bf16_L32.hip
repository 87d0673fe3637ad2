// Instantiations of the register-staged projection kernel, bf16, 32-row x 512-word tile.
#include "k1_stage.hpp"

namespace kb {
hipError_t launch_k1_stage_bf16_L32(int kc, dim3 grid, const K1Args& a, hipStream_t st) {
  return launch_k1_stage<LayL32, false>(kc, grid, a, st);
}
}  // namespace kb
