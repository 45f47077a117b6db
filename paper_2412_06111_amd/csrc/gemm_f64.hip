// The generic contraction with FP64 operands (gemm_tile.hpp).
#include "gemm_tile.hpp"

namespace ttnn {

TileKernels tile_kernels_f64() {
  return TileKernels{launch_tiles<double>, launch_tiles_lin<double>, reinterpret_cast<const void*>(ingest_kernel<double>)};
}

}  // namespace ttnn
