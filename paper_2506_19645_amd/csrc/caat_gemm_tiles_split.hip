// Tiles of the grouped bf16 shard GEMM whose contraction two groups of waves share.
#include "caat_gemm_tiles.h"

namespace caat {
CAAT_INSTANTIATE_TILES(Cfg128x128k)
CAAT_INSTANTIATE_TILES(Cfg64x64k)
}  // namespace caat
