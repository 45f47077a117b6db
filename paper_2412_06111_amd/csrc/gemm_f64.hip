// The generic contraction with FP64 operands (gemm_tile.hpp).
#include "gemm_tile.hpp"

namespace ttnn {

TileKernels tile_kernels_f64() {
  return TileKernels{launch_tiles<true, double>, launch_tiles<false, double>,
                     reinterpret_cast<const void*>(ingest_kernel<double>)};
}

}  // namespace ttnn
