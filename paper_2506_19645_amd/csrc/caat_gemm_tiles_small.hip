// 64 x 128 and 64 x 64 tiles of the grouped bf16 shard GEMM.
#include "caat_gemm_tiles.h"

namespace caat {
CAAT_INSTANTIATE_TILES(Cfg64x128)
CAAT_INSTANTIATE_TILES(Cfg64x64)
}  // namespace caat
