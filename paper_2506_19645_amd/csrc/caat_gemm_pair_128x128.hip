// Pairs of GEMMs in one launch, 128 x 128 tiles.
#include "caat_gemm_tiles.h"

namespace caat {
CAAT_INSTANTIATE_PAIR(Cfg128x128)
}  // namespace caat
