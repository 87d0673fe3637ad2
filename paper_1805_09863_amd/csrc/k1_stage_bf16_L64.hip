// Instantiations of the register-staged projection kernel, bf16, 64-row x 256-word tile.
#include "k1_stage.hpp"

namespace kb {
hipError_t launch_k1_stage_bf16_L64M(int kc, dim3 grid, const K1Args& a, hipStream_t st) {
  return launch_k1_stage<LayL64M, false>(kc, grid, a, st);
}
}  // namespace kb
