// Pairs of GEMMs in one launch, 256 x 256 tiles.
#include "caat_gemm_tiles.h"

namespace caat {
CAAT_INSTANTIATE_PAIR(Cfg256x256)
}  // namespace caat
