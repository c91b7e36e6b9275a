// 256 x 256 tiles of the grouped bf16 shard GEMM.
#include "caat_gemm_tiles.h"

namespace caat {
CAAT_INSTANTIATE_TILES(Cfg256x256)
}  // namespace caat
