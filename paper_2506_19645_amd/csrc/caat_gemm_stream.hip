// Instantiations and tile choice of the weight-streaming GEMM (kernel template in caat_gemm_stream.h).
#include "caat_gemm_stream.h"

namespace caat {

template <int MT, int RT, int NW, int LDS_KB, int EPI>
static hipError_t stream_launch(const GemmParams& p, hipStream_t s) {
  const long long tiles = (long long)((p.M + MT * 16 - 1) / (MT * 16)) * ((p.N + p.bn_out - 1) / p.bn_out) * p.G;
  if (tiles <= 0 || tiles > 0x7FFFFFFFLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((gemm_stream_kernel<MT, RT, NW, LDS_KB, EPI>), dim3((unsigned)tiles), dim3(64 * NW), 0, s, p);
  return hipGetLastError();
}

// Widths a workgroup may cover: RT tiles of 16 weight rows per MT tiles of 16 token rows, with the LDS that gives every
// wave two slots or more and, for few token rows, two or three workgroups per compute unit.
template <int EPI>
static hipError_t stream_plain(const GemmParams& p, const StreamTile& t, hipStream_t s) {
  switch (t.mt * 8 + t.rt) {
    case 8 + 2: return t.two_waves ? stream_launch<1, 2, 2, 24, EPI>(p, s) : stream_launch<1, 2, 4, 48, EPI>(p, s);
    case 8 + 3: return stream_launch<1, 3, 4, 64, EPI>(p, s);
    case 8 + 4: return t.two_waves ? stream_launch<1, 4, 2, 40, EPI>(p, s) : stream_launch<1, 4, 4, 80, EPI>(p, s);
    case 16 + 2: return stream_launch<2, 2, 4, 64, EPI>(p, s);
    case 16 + 3: return stream_launch<2, 3, 4, 80, EPI>(p, s);
    case 16 + 4: return stream_launch<2, 4, 4, 96, EPI>(p, s);
    case 24 + 2: return stream_launch<3, 2, 4, 80, EPI>(p, s);
    case 24 + 3: return stream_launch<3, 3, 4, 96, EPI>(p, s);
    case 24 + 6: return stream_launch<3, 6, 4, 144, EPI>(p, s);
    case 32 + 2: return stream_launch<4, 2, 4, 96, EPI>(p, s);
    case 32 + 3: return stream_launch<4, 3, 4, 112, EPI>(p, s);
    case 32 + 4: return stream_launch<4, 4, 4, 128, EPI>(p, s);
    case 32 + 6: return stream_launch<4, 6, 4, 160, EPI>(p, s);
    default: return hipErrorInvalidValue;
  }
}
static hipError_t stream_swiglu(const GemmParams& p, const StreamTile& t, hipStream_t s) {
  switch (t.mt * 8 + t.rt) {
    case 8 + 2: return stream_launch<1, 2, 4, 48, EPI_SWIGLU_FWD>(p, s);
    case 16 + 2: return stream_launch<2, 2, 4, 64, EPI_SWIGLU_FWD>(p, s);
    case 16 + 4: return stream_launch<2, 4, 4, 96, EPI_SWIGLU_FWD>(p, s);
    case 16 + 6: return stream_launch<2, 6, 4, 128, EPI_SWIGLU_FWD>(p, s);
    case 24 + 2: return stream_launch<3, 2, 4, 80, EPI_SWIGLU_FWD>(p, s);
    case 24 + 4: return stream_launch<3, 4, 4, 112, EPI_SWIGLU_FWD>(p, s);
    case 24 + 6: return stream_launch<3, 6, 4, 144, EPI_SWIGLU_FWD>(p, s);
    case 32 + 2: return stream_launch<4, 2, 4, 96, EPI_SWIGLU_FWD>(p, s);
    case 32 + 4: return stream_launch<4, 4, 4, 128, EPI_SWIGLU_FWD>(p, s);
    case 32 + 6: return stream_launch<4, 6, 4, 160, EPI_SWIGLU_FWD>(p, s);
    default: return hipErrorInvalidValue;
  }
}

StreamTile choose_stream_tile(const GemmParams& p, int epilogue, int n_cu) {
  const bool swi = epilogue == EPI_SWIGLU_FWD;
  const int m16 = (p.M + 15) / 16, tiles_m = (m16 + 3) / 4, mt = (m16 + tiles_m - 1) / tiles_m;
  // a wave should have some chunks of k: with fewer than 18 chunks of 64 two waves share a workgroup's contraction (us, two
  // waves / four: K = 512, 1 token row, 33 MB 8.4 / 10.4; K = 1024, 16 rows, 134 MB 25.0 / 26.9; K = 1376, 1 row, 90 MB
  // 21.5 / 19.0)
  StreamTile t = {mt, 0, 0, !swi && mt == 1 && (p.K + 63) / 64 < 18, 0};
  // A launch takes as long as the compute unit with the most rows to read: the weight rows of a tile plus its token
  // rows (from L2, at about a third of the cost), times the tiles a compute unit gets.
  static const int plain_rt[4][4] = {{2, 3, 4, 0}, {2, 3, 4, 0}, {2, 3, 6, 0}, {2, 3, 4, 6}};
  static const int swiglu_rt[4][4] = {{2, 0, 0, 0}, {2, 4, 6, 0}, {2, 4, 6, 0}, {2, 4, 6, 0}};
  double best = 0.0;
  for (int i = 0; i < 4; ++i) {
    const int rt = swi ? swiglu_rt[mt - 1][i] : plain_rt[mt - 1][i];
    if (rt == 0 || (t.two_waves && rt == 3)) continue;
    const int full = (swi ? rt / 2 : rt) * 16;
    for (int bn = full; bn > full - 16; bn -= 8) {
      const long long tiles = (long long)tiles_m * (((long long)p.N + bn - 1) / bn) * p.G;
      const double cost = (double)((tiles + n_cu - 1) / n_cu) * ((swi ? 2 : 1) * bn + 0.3 * 16 * mt);
      if (t.rt == 0 || cost < best) {
        best = cost;
        t.rt = rt;
        t.bn = bn;
        t.tiles = tiles;
      }
    }
  }
  return t;
}

hipError_t launch_gemm_stream(const GemmParams& p, int epilogue, int n_cu, hipStream_t s) {
  const StreamTile t = choose_stream_tile(p, epilogue, n_cu);
  GemmParams q = p;
  q.bn_out = t.bn;
  switch (epilogue) {
    case EPI_PLAIN: return stream_plain<EPI_PLAIN>(q, t, s);
    case EPI_GELU_FWD: return stream_plain<EPI_GELU_FWD>(q, t, s);
    case EPI_ROWPAR: return stream_plain<EPI_ROWPAR>(q, t, s);
    case EPI_SWIGLU_FWD: return stream_swiglu(q, t, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace caat
