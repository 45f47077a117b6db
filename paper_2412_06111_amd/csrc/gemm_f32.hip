// The generic contraction with FP32 operands (gemm_tile.hpp).
#include "gemm_tile.hpp"

namespace ttnn {

TileKernels tile_kernels_f32() {
  return TileKernels{launch_tiles<float>, launch_tiles_lin<float>, reinterpret_cast<const void*>(ingest_kernel<float>)};
}

}  // namespace ttnn
