// Instantiations of the direct projection kernel, bf16.
#include "k1_direct.hpp"

namespace kb {
hipError_t launch_k1_direct_bf16(int layout, int kc, dim3 grid, const K1Args& a, hipStream_t st) {
  switch (layout) {
    case K1_L128: return launch_k1_direct<LayL128, false>(kc, grid, a, st);
    case K1_L32: return launch_k1_direct<LayL32, false>(kc, grid, a, st);
    case K1_L32S: return launch_k1_direct<LayL32S, false>(kc, grid, a, st);
    default: return hipErrorInvalidValue;
  }
}
}  // namespace kb
