// The block-sized tile shapes of the grouped bf16 shard GEMM and their launch: every (layout, epilogue) pair that exists,
// instantiated per shape in the caat_gemm_tiles_*.hip units.
#pragma once
#include "caat_gemm_kernel.h"

namespace caat {

// 256 x 256: 8 waves, two stages of 64 k, one persistent workgroup per compute unit (stages of 32 k fetch an operand that is
// contiguous along K in 64-byte pieces of rows that lie kilobytes apart and meet at twice as many barriers: with five of
// them and the two halves of a line copied back to back, NT 241 us against 210, TN 210 against 203).
typedef TileCfg<256, 256, 2, 4, 2, true> Cfg256x256;
typedef TileCfg<192, 256, 2, 4, 2, true> Cfg192x256;
typedef TileCfg<256, 192, 4, 2, 2, true> Cfg256x192;
typedef TileCfg<128, 128, 2, 2, 2, false> Cfg128x128;   // two workgroups per compute unit
typedef TileCfg<64, 128, 2, 2, 3, false> Cfg64x128;     // two workgroups per compute unit
typedef TileCfg<64, 64, 2, 2, 4, false> Cfg64x64;       // two workgroups per compute unit
typedef TileCfg<128, 128, 2, 2, 2, false, false, 2> Cfg128x128k;   // two groups of four waves share the contraction (NN, TN)
typedef TileCfg<64, 64, 2, 2, 4, false, false, 2> Cfg64x64k;

template <class CFG>
hipError_t launch_block_sized(const GemmParams& p, int layout, int epilogue, hipStream_t s);

// two GEMMs in one launch: epilogue1 EPI_PLAIN, EPI_GELU_BWD or EPI_SWIGLU_BWD: p1 NN, p2 TN and plain; EPI_ROWPAR: both NT, p2
// with EPI_PARTIAL or EPI_SHARED_BCAST
template <class CFG>
hipError_t launch_pair(const GemmPair& pair, const GemmParams& p1, int epilogue1, const GemmParams& p2, int epilogue2,
                       const NormSums& sums, hipStream_t s);

template <class CFG>
static hipError_t launch_pair_impl(const GemmPair& pair, const GemmParams& p1, int epilogue1, const GemmParams& p2, int epilogue2,
                                   const NormSums& sums, hipStream_t s) {
  typedef GemmKind<true, true, EPI_PLAIN> Wgrad;
  typedef GemmKind<false, false, EPI_ROWPAR> Private;
  if (epilogue1 == EPI_ROWPAR) {
    if (epilogue2 == EPI_PARTIAL) return launch_pair_one<CFG, Private, GemmKind<false, false, EPI_PARTIAL>>(pair, p1, p2, sums, s);
    if (epilogue2 == EPI_SHARED_BCAST) return launch_pair_one<CFG, Private, GemmKind<false, false, EPI_SHARED_BCAST>>(pair, p1, p2, sums, s);
    return hipErrorInvalidValue;
  }
  if (epilogue2 != EPI_PLAIN) return hipErrorInvalidValue;
  switch (epilogue1) {
    case EPI_PLAIN: return launch_pair_one<CFG, GemmKind<false, true, EPI_PLAIN>, Wgrad>(pair, p1, p2, sums, s);
    case EPI_GELU_BWD: return launch_pair_one<CFG, GemmKind<false, true, EPI_GELU_BWD>, Wgrad>(pair, p1, p2, sums, s);
    case EPI_SWIGLU_BWD: return launch_pair_one<CFG, GemmKind<false, true, EPI_SWIGLU_BWD>, Wgrad>(pair, p1, p2, sums, s);
    default: return hipErrorInvalidValue;
  }
}

#define CAAT_INSTANTIATE_PAIR(CFG)                                                                                             \
  template <>                                                                                                                  \
  hipError_t launch_pair<CFG>(const GemmPair& pair, const GemmParams& p1, int epilogue1, const GemmParams& p2, int epilogue2,  \
                              const NormSums& sums, hipStream_t s) {                                                           \
    return launch_pair_impl<CFG>(pair, p1, epilogue1, p2, epilogue2, sums, s);                                                 \
  }

#define CAAT_INSTANTIATE_TILES(CFG)                                                                                            \
  template <>                                                                                                                  \
  hipError_t launch_block_sized<CFG>(const GemmParams& p, int layout, int epilogue, hipStream_t s) {                           \
    return launch_block_sized_impl<CFG>(p, layout, epilogue, s);                                                               \
  }

template <class CFG>
static hipError_t launch_block_sized_impl(const GemmParams& p, int layout, int epilogue, hipStream_t s) {
  switch (layout) {
    case 0:  // NT
      if constexpr (CFG::KW > 1) return hipErrorInvalidValue;   // (see choose_tile)
      else switch (epilogue) {
        case EPI_PLAIN: return launch_one<CFG, false, false, EPI_PLAIN>(p, s);
        case EPI_GELU_FWD: return launch_one<CFG, false, false, EPI_GELU_FWD>(p, s);
        case EPI_SWIGLU_FWD:   // a wave needs its 32 gate and 32 up columns side by side
          if constexpr (CFG::WTN % 64 == 0) return launch_one<CFG, false, false, EPI_SWIGLU_FWD>(p, s);
          else return hipErrorInvalidValue;
        case EPI_ROWPAR: return launch_one<CFG, false, false, EPI_ROWPAR>(p, s);
        case EPI_SHARED_BCAST: return launch_one<CFG, false, false, EPI_SHARED_BCAST>(p, s);
        case EPI_PARTIAL: return launch_one<CFG, false, false, EPI_PARTIAL>(p, s);
        case EPI_ROPE:         // see gemm_takes_rope
          if constexpr (CFG::WTN == 64) return launch_one<CFG, false, false, EPI_ROPE>(p, s);
          else return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
      }
    case 1:  // NN
      switch (epilogue) {
        case EPI_PLAIN: return launch_one<CFG, false, true, EPI_PLAIN>(p, s);
        case EPI_GELU_BWD: return launch_one<CFG, false, true, EPI_GELU_BWD>(p, s);
        case EPI_SWIGLU_BWD: return launch_one<CFG, false, true, EPI_SWIGLU_BWD>(p, s);
        default: return hipErrorInvalidValue;
      }
    case 2:  // TN
      if (epilogue == EPI_PLAIN) return launch_one<CFG, true, true, EPI_PLAIN>(p, s);
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

}  // namespace caat
