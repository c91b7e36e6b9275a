// Pairs of GEMMs in one launch, 64 x 128 and 64 x 64 tiles.
#include "caat_gemm_tiles.h"

namespace caat {
CAAT_INSTANTIATE_PAIR(Cfg64x128)
CAAT_INSTANTIATE_PAIR(Cfg64x64)
}  // namespace caat
