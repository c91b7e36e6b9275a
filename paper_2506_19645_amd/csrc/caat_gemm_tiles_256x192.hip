// 256 x 192 tiles of the grouped bf16 shard GEMM.
#include "caat_gemm_tiles.h"

namespace caat {
CAAT_INSTANTIATE_TILES(Cfg256x192)
}  // namespace caat
