// The generic contraction with BF16 operands (gemm_tile.hpp).
#include "gemm_tile.hpp"

namespace ttnn {

TileKernels tile_kernels_bf16() {
  return TileKernels{launch_tiles<uint16_t>, launch_tiles_lin<uint16_t>, reinterpret_cast<const void*>(ingest_kernel<uint16_t>)};
}

}  // namespace ttnn
