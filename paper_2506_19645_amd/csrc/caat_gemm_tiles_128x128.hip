// 128 x 128 tiles of the grouped bf16 shard GEMM.
#include "caat_gemm_tiles.h"

namespace caat {
CAAT_INSTANTIATE_TILES(Cfg128x128)
}  // namespace caat
