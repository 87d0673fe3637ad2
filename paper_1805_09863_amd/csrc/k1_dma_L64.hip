// Instantiations of the DMA-pipelined bf16 projection kernel, layout L64.
#include "k1_dma.hpp"

namespace kb {
hipError_t launch_k1_dma_L64(int kc, dim3 grid, const K1Args& a, hipStream_t st) {
  return launch_k1_dma_layout<LayL64>(kc, grid, a, st);
}
hipError_t launch_k1_dma_L64M(int kc, dim3 grid, const K1Args& a, hipStream_t st) {
  return launch_k1_dma_layout<LayL64M>(kc, grid, a, st);
}
}  // namespace kb
