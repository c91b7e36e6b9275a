// Instantiations and launch dispatch of the grouped bf16 shard GEMM (kernel template in caat_gemm_kernel.h).
#include <algorithm>
#include <cmath>
#include "caat_gemm_tiles.h"

namespace caat {

typedef TileCfg<64, 128, 2, 2, 4, false, true> CfgSkinny;   // small batches whose weights fill the chip

// the specialisations live in the caat_gemm_tiles_*.hip units
template <> hipError_t launch_block_sized<Cfg256x256>(const GemmParams&, int, int, hipStream_t);
template <> hipError_t launch_block_sized<Cfg192x256>(const GemmParams&, int, int, hipStream_t);
template <> hipError_t launch_block_sized<Cfg256x192>(const GemmParams&, int, int, hipStream_t);
template <> hipError_t launch_block_sized<Cfg128x128>(const GemmParams&, int, int, hipStream_t);
template <> hipError_t launch_block_sized<Cfg64x128>(const GemmParams&, int, int, hipStream_t);
template <> hipError_t launch_block_sized<Cfg64x64>(const GemmParams&, int, int, hipStream_t);
template <> hipError_t launch_block_sized<Cfg128x128k>(const GemmParams&, int, int, hipStream_t);
template <> hipError_t launch_block_sized<Cfg64x64k>(const GemmParams&, int, int, hipStream_t);

#define CAAT_PAIR(CFG) \
  template <> hipError_t launch_pair<CFG>(const GemmPair&, const GemmParams&, int, const GemmParams&, int, const NormSums&, hipStream_t);
CAAT_PAIR(Cfg256x256) CAAT_PAIR(Cfg192x256) CAAT_PAIR(Cfg128x128) CAAT_PAIR(Cfg64x128) CAAT_PAIR(Cfg64x64)
#undef CAAT_PAIR

int compute_units() {
  static int n_cu = 0;
  if (n_cu == 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess)
      n_cu = v;
    if (n_cu <= 0) n_cu = 256;
  }
  return n_cu;
}

// Output columns a 64 x 128 tile covers (a multiple of 8 up to the tile's width): what a compute unit can have in flight
// is bounded, so the time is set by the bytes it has to pull, per tile the weight rows it covers (from HBM) plus the 64
// activation rows every tile re-reads (from L2, at about a third of the latency: counted as 20 rows), times the tiles a
// compute unit gets.  The width that minimises this, the widest on a tie.
static int choose_skinny_width(int G, int N, int epilogue) {
  const int full = epilogue == EPI_SWIGLU_FWD ? CfgSkinny::BN / 2 : CfgSkinny::BN;
  const int n_cu = compute_units();
  int width = full;
  long long best = -1;
  for (int bn = full; bn >= 16; bn -= 8) {
    const long long tiles = (long long)((N + bn - 1) / bn) * G;
    const long long cost = ((tiles + n_cu - 1) / n_cu) * ((epilogue == EPI_SWIGLU_FWD ? 2 : 1) * bn + 20);
    if (best < 0 || cost < best) {
      best = cost;
      width = bn;
    }
  }
  return width;
}

// Tile shape of a block-sized launch: the one with the least modelled time.  A launch runs in rounds of as many tiles as
// the compute units hold at once; a tile takes a time per 64-k stage and a fixed time (its first stages, its epilogue),
// and a round that leaves compute units idle is faster than a full one (clock, caches), down to 0.55 of its time.  The
// constants are fitted to the shapes of some training and prefill blocks, all three layouts, 40 launches from 150 to 8192
// rows timed with every tile shape: the choice by the model is 0.4 % slower than the fastest shape on their average.
// On 7075 other launches, sizes drawn at random, it is 0.8 % slower on average; 2 % of them, most with rows that are no whole
// 128-byte lines or few stages of k, are more than 10 % off, 41 % at worst (NT 2 x 6890 x 88 x 6776).  Constants fitted to
// half of these, with a cost for such rows and a least fill for each shape, still leave the other half 0.7 % off.
// The last two shapes share a tile's contraction between two groups of four waves: for launches with a tile or less per
// compute unit, whose time is the chain of stages and not the matrix unit.  They are for the gradients only (NN, TN): a
// tile of the forward pass (NT) is one sum in ascending k whatever its shape, so that a channel's bits are the same with
// the reduce inside the GEMM and as a pass of its own (for 65 to 128 rows see choose_route).
// Examples (us; 256 x 256, 192 x 256, 256 x 192, 128 x 128, 64 x 128, 64 x 64, 128 x 128 and 64 x 64 shared; G x M x N x K):
//   NT 8 x 777 x 1536 x 4096     111 /  99 /  99 / 123 / 123 / 153 / 124 / 172
//   TN 4 x 2048 x 1408 x 1111   34.4 / 50.3 / 31.4 / 38.8 / 42.2 / 56.2 / 46.6 / 73.2
//   NN 4 x 1111 x 1408 x 2048   49.0 / 40.9 / 44.4 / 33.5 / 45.3 / 57.7 / 46.2 / 68.9
//   TN 4 x 2048 x 512 x 3009    68.4 / 58.6 / 61.1 / 39.0 / 38.0 / 49.7 / 32.7 / 56.3
//   NT 2 x 256 x 768 x 1536     33.7 / 28.8 / 29.0 / 19.6 / 13.1 / 11.2 / 16.2 /  9.9
//   NN 2 x 256 x 768 x 1536     34.7 / 29.1 / 31.3 / 19.2 / 13.9 / 12.0 / 16.2 / 10.0
//   NN 8 x 500 x 768 x 3072     67.6 / 59.0 / 64.7 / 39.3 / 34.7 / 42.8 / 32.3 / 44.4
//   NN 4 x 8192 x 2048 x 2048    227 /  256 /  260 /  275 /  369 /  479
// 128 x 256 and 256 x 128 tiles with three stages came within 5 % of the best of these wherever they won, and 256 x 256
// by four waves of 128 x 128 (a third less LDS traffic, one wave per SIMD) takes 15 % longer than by eight.
struct TileShape {
  int bm, bn, per_cu;   // per_cu: workgroups a compute unit holds
  int k;                // depth of a stage
  double stage, tile;   // us
  bool persist;
};
static constexpr TileShape TILES[] = {{256, 256, 1, 64, 1.64, 8.1, true}, {192, 256, 1, 64, 1.35, 6.3, true},
                                      {256, 192, 1, 64, 1.35, 6.7, true}, {128, 128, 2, 64, 0.98, 4.2, false},
                                      {64, 128, 2, 64, 0.69, 2.6, false}, {64, 64, 2, 64, 0.446, 1.8, false},
                                      {128, 128, 1, 128, 1.15, 3.8, false}, {64, 64, 1, 128, 0.473, 2.5, false}};
static int choose_tile(const GemmParams& p, int layout, int epilogue, int n_cu, double* us = nullptr) {
  const bool swi = epilogue == EPI_SWIGLU_FWD;
  int best = 0;
  double cost = 0.0;
  for (int i = 0; i < (int)(sizeof(TILES) / sizeof(TILES[0])); ++i) {
    const TileShape& t = TILES[i];
    if (swi && (t.bn == 192 || t.bn == 64)) continue;   // a wave takes gate and up columns in pairs of 32
    if (layout == 0 && t.k > 64) continue;
    const long long bn_out = swi ? t.bn / 2 : t.bn, slots = (long long)t.per_cu * n_cu;
    const long long tiles = (((long long)p.M + t.bm - 1) / t.bm) * ((p.N + bn_out - 1) / bn_out) * p.G;
    const long long full = tiles / slots, rest = tiles % slots;
    const double rounds = (double)full + (rest ? 0.55 + 0.45 * (double)rest / (double)slots : 0.0);
    const double nk = (double)(((long long)p.K + t.k - 1) / t.k) * (p.kcat > 1 ? p.kcat : 1);
    const double c = rounds * (nk * t.stage + t.tile);
    if (i == 0 || c < cost) {
      cost = c;
      best = i;
    }
  }
  if (us) *us = cost;
  return best;
}

// Few token rows (NT): the weights are what has to be read.  The streaming kernel reads them best, except where many token
// rows meet many weight rows: every workgroup reads all of its token rows, so there a tile kernel takes over (the 64 x 128
// one up to 64 token rows).  Weight rows whose stride is a multiple of 4 KB start on the same memory channels; the tiles, which
// read a piece of 128 rows at a time, lose 5 to 30 % by that, and the line lies higher.  Streaming / tile kernel, us, weights from
// HBM; the lines from 17 to 64 rows are chosen on 2810 products with 24 to 64 token rows each (512 to 8192 k, 30 to 128 weight rows
// per compute unit, 2 to 8 ranks): 0.3 % off the fastest kernel on average, 23 % at worst.
//   1 - 16    always, but for SwiGLU with 65 to 80 and 97 to 112 weight rows per compute unit (stride of 4 KB: always): tiles of
//             16 gate and 16 up rows take three and four rounds, 64 x 128 tiles one.  1 / 16 token rows: 28672 of 5120 52.7 / 59.1
//             against 45.2 / 45.9, 28672 of 512 12.2 / 12.3 against 8.4 / 8.6; at 81 to 96 and 113 to 128 the tiles gain 5 % at best
//   17 - 32   below 80 weight rows per compute unit (stride of 4 KB: 128).  32 token rows: 20480 of 1728 16.2 / 15.9, 27648 of 5120
//             55 / 49, 28672 of 8192 79 / 91, of 4096 45.0 / 47.5
//   33 - 64   below 65 (stride of 4 KB: 96).  48 token rows: 20480 of 1728 17.4 / 16.4, 27648 of 5120 61 / 50, 22016 of 4096
//             36.6 / 38.8, 28672 of 4096 48.0 / 47.0 (in a layer 48.6 / 45.8); 64 token rows: 20480 of 1728 19.4 / 16.6, 24576 of
//             2048 25.0 / 23.9, 22016 of 4096 38.0 / 38.6
//   33 - 48   leave the streaming kernel no good tile for 49 to 64 weight rows per compute unit, which is one 64 x 64 tile for
//             each: 48 token rows, streaming / 64 x 64: 13824 of 5120 39.2 / 33.1, 15360 of 5120 39.3 / 33.2, 16384 of 1376
//             15.8 / 14.2; stride of 4 KB: 16384 of 6144 47.0 / 46.3, no gain on average; 56 rows 13824 of 5120 32.2 / 33.4
//   65 - 128  while one round of workgroups covers the launch, or two of the widest a long contraction.  96 token rows, one
//             round: 6144 of 4096 17.1 / 24.2, 12288 of 4096 28.4 / 36.8; two of the widest: 20480 of 1728 28.9 / 27.7, 24576 of
//             2048 33.9 / 33.2, 22016 of 4096 56.8 / 57.8 (in a layer 61.0 / 63.2); other: 8192 of 5504 35.7 / 33.6, 16384 of
//             1376 25.7 / 20.8, 28672 of 4096 75.7 / 62.3, 32768 of 512 23.7 / 12.8, but 18432 of 6144 76 / 88
// The streaming kernel adds up sums of several waves, the tiles are one sum.  So a row-parallel GEMM on the private columns
// of a shard alone (reduce_in_gemm, more than 64 rows) goes by the columns of the whole shard, as without reduce_in_gemm.
enum { ROUTE_FEW_ROWS = 8, ROUTE_STREAM = 16 };
static int choose_route(const GemmParams& p, int layout, int epilogue, int n_cu) {
  if (layout == 0 && p.M <= 128 && epilogue != EPI_SHARED_BCAST && epilogue != EPI_PARTIAL) {
    GemmParams q = p;
    if (p.n_route > 0) q.N = p.n_route;
    const long long wrows = (long long)q.G * q.N * (epilogue == EPI_SWIGLU_FWD ? 2 : 1);
    const StreamTile t = choose_stream_tile(q, epilogue, n_cu);
    const bool pages = p.K % 2048 == 0;   // rows of whole 4 KB
    bool stream = true;
    if (p.M > 64) stream = t.tiles <= n_cu || (t.tiles <= 2LL * n_cu && t.rt == 6 && p.K >= 4096);
    else if (p.M <= 16) stream = !(epilogue == EPI_SWIGLU_FWD && !pages && ((wrows > 64LL * n_cu && wrows <= 80LL * n_cu) ||
                                                                           (wrows > 96LL * n_cu && wrows <= 112LL * n_cu)));
    else stream = wrows < (p.M <= 32 ? (pages ? 128LL : 80LL) : (pages ? 96LL : 65LL)) * n_cu;
    const bool one_tile_each = p.M > 32 && p.M <= 48 && !pages && wrows > 48LL * n_cu && wrows <= 64LL * n_cu &&
                               epilogue != EPI_SWIGLU_FWD;
    if (stream && !one_tile_each) return ROUTE_STREAM;
    if (p.M <= 64 && !one_tile_each) return ROUTE_FEW_ROWS;
  }
  return choose_tile(p, layout, epilogue, n_cu);
}

static bool in_range(const GemmParams& p, int epilogue) {
  // buffer-load offsets are 32-bit and relative to the tile origin: the farthest row a tile touches times the
  // row stride must stay below 2 GiB
  const long long far_rows = (epilogue == EPI_SWIGLU_FWD ? (long long)p.half : 0) + 256 + 64;  // rows or k-rows
  if (far_rows * p.lda * 2 >= 0x7FFFF000LL || far_rows * p.ldb * 2 >= 0x7FFFF000LL) return false;
  // the epilogue's buffer offsets are relative to a wave's first row: up to 256 rows of any output / second operand
  const long long ldmax = std::max(std::max(p.ldc, p.ldc2), p.ldaux);
  const long long elem = epilogue == EPI_PARTIAL ? 4 : 2;
  return (256 * ldmax + 2 * (long long)p.half + (long long)p.N) * elem < 0x7FFFFFFFLL;
}

// Only where the plain product's own tile has waves of 64 columns, 32 channels of a head and the 32 that they are rotated with
// (256 x 256, 192 x 256, 128 x 128, 64 x 128); 256 x 192 and 64 x 64 tiles and the kernels for few rows leave the rotation to a
// pass of its own, whose time the choice of another tile would cost.  With the pass / in the epilogue, forward and backward of an
// attention block of h = 4096, T = 8, 4096 tokens 2455 / 2418 us, 3 x 1003 tokens of 2048, T = 4, 8 key heads 454 / 446; a
// prefill layer of 16 x 2048 tokens of 4096 15.37 / 15.21 ms, of 777 464.7 / 460.8 us.
// Nor 256 x 256 tiles with sequences of fewer than 8 tokens: every sine and cosine is then taken anew in each of a wave's eight
// steps of 16 rows, which a full chip of large tiles does not hide.  Forward passes on such tiles, time with the pass over time in
// the epilogue, 1335 random blocks and layers: 1 token 0.987 (worst 0.942), 2 0.991, 3 0.998, 4 and 5 1.003 (worst 0.971), 6 and 7
// 1.001, 8 to 11 1.010, 12 to 31 1.010, 128 and more 1.023; on 192 x 256 tiles 1.001 at 1 token, 1.01 to 1.08 from 2 tokens on
// the others.
bool gemm_takes_rope(const GemmParams& p) {
  const int r = choose_route(p, 0, EPI_PLAIN, compute_units());
  if (r == 0 && p.rope.seq < 8) return false;
  return (r == 0 || r == 1 || r == 3 || r == 4) && in_range(p, EPI_PLAIN);
}

hipError_t launch_gemm(const GemmParams& p, int layout, int epilogue, hipStream_t s) {
  if (!in_range(p, epilogue)) return hipErrorInvalidValue;
  if (epilogue == EPI_ROPE && (layout != 0 || !gemm_takes_rope(p))) return hipErrorInvalidValue;
  const int n_cu = compute_units();
  GemmParams q = p;
  q.bn_out = 0;  // block-sized tiles always cover their full width
  switch (choose_route(p, layout, epilogue == EPI_ROPE ? (int)EPI_PLAIN : epilogue, n_cu)) {
    case 0: return launch_block_sized<Cfg256x256>(q, layout, epilogue, s);
    case 1: return launch_block_sized<Cfg192x256>(q, layout, epilogue, s);
    case 2: return launch_block_sized<Cfg256x192>(q, layout, epilogue, s);
    case 3: return launch_block_sized<Cfg128x128>(q, layout, epilogue, s);
    case 4: return launch_block_sized<Cfg64x128>(q, layout, epilogue, s);
    case 5: return launch_block_sized<Cfg64x64>(q, layout, epilogue, s);
    case 6: return launch_block_sized<Cfg128x128k>(q, layout, epilogue, s);
    case 7: return launch_block_sized<Cfg64x64k>(q, layout, epilogue, s);
    case ROUTE_STREAM: return launch_gemm_stream(p, epilogue, n_cu, s);
    default: break;
  }
  q.bn_out = choose_skinny_width(p.G, p.N, epilogue);
  switch (epilogue) {
    case EPI_PLAIN: return launch_one<CfgSkinny, false, false, EPI_PLAIN>(q, s);
    case EPI_GELU_FWD: return launch_one<CfgSkinny, false, false, EPI_GELU_FWD>(q, s);
    case EPI_SWIGLU_FWD: return launch_one<CfgSkinny, false, false, EPI_SWIGLU_FWD>(q, s);
    case EPI_ROWPAR: return launch_one<CfgSkinny, false, false, EPI_ROWPAR>(q, s);
    default: return hipErrorInvalidValue;
  }
}

// What a tile's stores to all ranks, and the loads of what is added to them, take at a compute unit's share of the copy rate: a
// launch of few large tiles ends with that (T = 16, 4979 tokens, h = 512, hs = 328, K = 112: 194 us with 117 tiles of 128 x 128 in
// the pair, 154 apart on 468 of 64 x 64).
static double bcast_us(const TileShape& t, double copies) { return copies * t.bm * t.bn * 4.0 / 21e3; }

// Both gradient GEMMs in one launch (gemm_pair_kernel): the one with the longer tiles first, on as many workgroups as fit on the
// chip; the other one's workgroups start wherever a slot is or comes free, each with one tile or, persistent tiles with an even
// share of several, which saves 1.5 us a tile.  Time by the model of the tile choice: the end of the last tile.  The tiles that
// only win alone (256 x 192 and those that share a contraction) are left out.
// Measured on 44 training steps of 135 to 8192 tokens, T = 2 to 8, h = 512 to 4096 (backward pass, us; one after the
// other / paired): 4 x 360 tokens of 512, ffn 1792 36.4 / 25.7, 8 x 147 of 1536, ffn 6144 57.8 / 41.2, 4 x 731 of 2048,
// ffn 5504 155 / 132, 4 x 1111 of 2048, ffn 5632 204 / 188, 4 x 8192 of 2048, ffn 8192 1027 / 1000.
// Two things the constants of single launches don't hold: 64 x 64 tiles beside another GEMM's take 10 % longer (3779 random pairs,
// each tile timed), and a GEMM of one row of persistent tiles pulls every byte of its weights from memory with one stage on its
// way, 1.4 times the time a stage takes from the caches (133 tokens of 4096, ffn 16384, T = 4: 230 us on 192 x 256 tiles, 205 apart).
static GemmPair plan_pair(const TileShape& t, int index, const GemmParams& p1, const GemmParams& p2, int n_cu, double copies) {
  auto tiles = [&](const GemmParams& p) { return (((long long)p.M + t.bm - 1) / t.bm) * (((long long)p.N + t.bn - 1) / t.bn) * p.G; };
  auto us = [&](const GemmParams& p) {
    const bool cold = t.persist && p.M <= t.bm && (&p == &p1 || p.kcat > 0);   // the weight gradient reads no weights
    const double stages = (double)(((long long)p.K + t.k - 1) / t.k) * (p.kcat > 1 ? p.kcat : 1);
    return stages * t.stage * (cold ? 1.4 : 1.0) + t.tile + (&p == &p2 ? bcast_us(t, copies) : 0.0);
  };
  const double u1 = us(p1), u2 = us(p2);
  const bool sf = u2 > u1;
  const long long slots = (long long)t.per_cu * n_cu, na = tiles(sf ? p2 : p1), nb = tiles(sf ? p1 : p2);
  const double ua = sf ? u2 : u1, ub = sf ? u1 : u2;
  // behind the first GEMM n_hi slots are free at hi, n_lo at lo
  const long long n_hi = na % slots, n_lo = slots - n_hi;
  const double lo = (double)(na / slots) * ua, hi = n_hi ? lo + ua : lo;
  // one tile at a time to whichever slot is free first: those free at lo catch up with the others, then whole rounds of all
  // slots, then the last tiles
  struct { double at; long long n; } cls[2] = {{lo, n_lo}, {hi, n_hi}};
  const double ub1 = ub + (t.persist ? 1.5 : 0.0);
  long long left = nb;
  const long long ahead = std::min(left / n_lo, (long long)((hi - lo) / ub1));
  cls[0].at += ahead * ub1;
  left -= ahead * n_lo;
  const long long rounds = left > 3 * slots ? left / slots - 2 : 0;
  left -= rounds * slots;
  cls[0].at += rounds * ub1;
  cls[1].at += rounds * ub1;
  while (left > 0) {
    const int c = cls[1].n && cls[1].at < cls[0].at ? 1 : 0;
    cls[c].at += ub1;
    left -= cls[c].n;
  }
  const double each = std::max(cls[0].at, n_hi ? cls[1].at : lo);
  double end = each;
  bool one_each = true;
  if (t.persist) {   // even shares: the first nb % g workgroups have one tile more
    const long long g = std::min(slots, nb), more = nb % g;
    const double share = (double)(nb / g) * ub;
    const double even = std::max({hi, lo + share + (more ? ub : 0.0), g > n_lo ? hi + share + (more > n_lo ? ub : 0.0) : 0.0});
    one_each = each < even;
    end = std::min(each, even);
  }
  const double fill = (na * ua + nb * ub) / (slots * end);
  return {index, sf, one_each, end * (0.55 + 0.45 * std::min(fill, 1.0)) * (t.bm == 64 && t.bn == 64 ? 1.1 : 1.0)};
}
static GemmPair best_pair(const GemmParams& p1, const GemmParams& p2, int n_cu, double copies = 0.0) {   // that p2 stores
  GemmPair best = {-1, false, false, 0.0};
  for (int i : {0, 1, 3, 4, 5}) {
    const GemmPair p = plan_pair(TILES[i], i, p1, p2, n_cu, copies);
    if (best.tile < 0 || p.us < best.us) best = p;
  }
  return best;
}
// A pair is taken if the model has it 2 % faster, or less than 4 us slower, that being what a launch less is worth; if all of it is
// the tile that both would take alone, a tie is a gain too (313 steps with such ties: 1.016 times as fast, worst 0.99 but for two).
// Of those 3779 pairs, each alone in a loop, 1.2 % then lose more than 2 %, and another 1.4 % of such ties; the average is 0.855 of
// the time apart (0.847 with the best choice for every one; "less than 2 us slower" for all: 3.1 %, 0.857).  Of 1873 backward
// passes 0.7 % lose more than 2 %, worst 0.925, average 1.153 times as fast.
static bool pays(double pair, double apart) { return pair < 0.98 * apart + 4.0; }
GemmPair gemm_pair(const GemmParams& nn, const GemmParams& tn) {
  const int n_cu = compute_units();
  GemmPair best = best_pair(nn, tn, n_cu);
  double a = 0.0, b = 0.0;
  const int ta = choose_tile(nn, 1, EPI_PLAIN, n_cu, &a), tb = choose_tile(tn, 2, EPI_PLAIN, n_cu, &b);
  if (!(ta == best.tile && tb == best.tile ? best.us < a + b + 2.0 : pays(best.us, a + b))) best.tile = -1;
  return best;
}

static hipError_t launch_any_pair(const GemmPair& p, const GemmParams& p1, int epilogue1, const GemmParams& p2, int epilogue2,
                                  const NormSums& sums, hipStream_t s) {
  if (!in_range(p1, epilogue1) || !in_range(p2, epilogue2)) return hipErrorInvalidValue;
  switch (p.tile) {
    case 0: return launch_pair<Cfg256x256>(p, p1, epilogue1, p2, epilogue2, sums, s);
    case 1: return launch_pair<Cfg192x256>(p, p1, epilogue1, p2, epilogue2, sums, s);
    case 3: return launch_pair<Cfg128x128>(p, p1, epilogue1, p2, epilogue2, sums, s);
    case 4: return launch_pair<Cfg64x128>(p, p1, epilogue1, p2, epilogue2, sums, s);
    case 5: return launch_pair<Cfg64x64>(p, p1, epilogue1, p2, epilogue2, sums, s);
    default: return hipErrorInvalidValue;
  }
}
hipError_t launch_gemm_pair(const GemmPair& p, const GemmParams& nn, int epilogue, const GemmParams& tn, const NormSums& sums,
                            hipStream_t s) {
  return launch_any_pair(p, nn, epilogue, tn, EPI_PLAIN, sums, s);
}

// The shared channels of all ranks as one product with a contraction kcat times as long: few tiles, each a long chain.
// A prompt of some hundred tokens leaves most of the chip idle, so the ranks are cut into groups that are summed in
// parallel into fp32 buffers, and a second kernel adds the groups up in ascending order.  The number of groups is the one
// with the least modelled time, the model of the tile choice (on the 256 compute units of the chip, so that
// the bits do not depend on the device that is current) times 1.4 for weights that come from HBM and not, as where the model was
// fitted, from the memory-side cache, plus the merge: 5 us and the fp32 sums at 7 TB/s.  Both constants are checked on 20
// products (2 to 8 ranks, h = 2048 to 8192, 512 to 5504 k per rank, hs = h / 2 and h / 4) of 65 to 2048 tokens: 0.4 % off the
// best number of groups on average, 11 % at worst.  Examples (us, 1 / 2 / 4 / 8 groups; tokens x hs x k per rank x ranks):
//   777 x 2048 x 512 x 8    40 / 41 / 40 / 45      777 x 2048 x 1376 x 8    117 / 91 / 66 / 67
//   65 x 2048 x 512 x 8     29 / 22 / 17 / 17     1024 x 2048 x 1376 x 8    112 / 93 / 80 / 72
//   777 x 1024 x 512 x 4    18 / 19 / 22           777 x 2048 x 3584 x 4    116 / 92 / 70
// `scratch_bytes`: what there is for the groups' sums.
static int gemm_shared_groups(int M, int N, int K, int kcat, size_t scratch_bytes) {
  GemmParams q = {};
  q.M = M;
  q.N = N;
  q.K = K;
  int best = 1;
  double cost = 0.0;
  for (int g = 1; g <= kcat; g *= 2) {
    if (kcat % g != 0 || (g > 1 && (size_t)g * M * N * sizeof(float) > scratch_bytes)) break;
    q.G = g;
    q.kcat = kcat / g;
    double us = 0.0;
    choose_tile(q, 0, EPI_PARTIAL, 256, &us);
    us *= 1.4;
    if (g > 1) us += 5.0 + (double)g * M * N * 4.0 / 7e6;
    if (g == 1 || us < cost) {
      cost = us;
      best = g;
    }
  }
  return best;
}

// As many groups as there are ranks, up to 128 MiB: does not fall when M grows, so that the scratch of the largest batch serves
// the smaller ones too.  By the model the limit costs nothing up to 8 ranks of K = 3584.
size_t gemm_shared_scratch_bytes(int M, int N, int kcat) {
  return kcat > 1 ? std::min((size_t)kcat * M * N * sizeof(float), (size_t)128 << 20) : 0;
}

// p cut into groups of ranks whose fp32 sums go to scratch
static GemmParams shared_groups(const GemmParams& p, int groups, void* scratch) {
  GemmParams q = p;
  q.G = groups;
  q.kcat = p.kcat / groups;
  q.stride_a = p.kstride_a * q.kcat;
  q.stride_b = p.kstride_b * q.kcat;
  q.c = reinterpret_cast<bf16_t*>(scratch);
  q.ldc = p.N;
  q.stride_c = (long long)p.M * p.N;
  q.aux = nullptr;
  q.ldaux = 0;
  return q;
}
static hipError_t merge_groups(const GemmParams& p, int groups, const void* scratch, hipStream_t s) {
  return launch_shared_merge(reinterpret_cast<const float*>(scratch), groups, p.aux, p.c, p.M, p.N, p.ldaux, p.ldc, p.stride_aux,
                             p.stride_c, p.bcast, s);
}
hipError_t launch_gemm_shared(const GemmParams& p, void* scratch, size_t scratch_bytes, hipStream_t s) {
  const int groups = gemm_shared_groups(p.M, p.N, p.K, p.kcat, scratch ? scratch_bytes : 0);
  if (groups == 1) return launch_gemm(p, 0, EPI_SHARED_BCAST, s);
  const hipError_t e = launch_gemm(shared_groups(p, groups, scratch), 0, EPI_PARTIAL, s);
  return e != hipSuccess ? e : merge_groups(p, groups, scratch, s);
}

// The private columns in the same launch: their tiles fill what the shared ones leave idle.  Not where they stream their weights
// (65 to 128 token rows, see choose_route).  The groups are those of the two launches, so the bits are the same either way.
// 681 random forward passes (1 to 16 ranks, 65 to 8192 tokens, h = 512 to 8192): 1.116 times as fast as one after the other, worst
// 0.972; 777 tokens of a 4096-channel layer, 8 ranks: 494 -> 481 us (474 with groups of its own, and other bits then).
GemmPair gemm_shared_pair(const GemmParams& p, const GemmParams& priv, size_t scratch_bytes, int* groups) {
  GemmPair pair = {-1, false, false, 0.0};
  const int n_cu = compute_units();
  double shared = 0.0, us = 0.0;
  *groups = gemm_shared_groups(p.M, p.N, p.K, p.kcat, scratch_bytes);
  if (choose_route(priv, 0, EPI_ROWPAR, n_cu) >= ROUTE_FEW_ROWS) return pair;
  const double copies = *groups == 1 ? (double)p.bcast : 0.0;
  GemmParams q = p;
  q.G = *groups;
  q.kcat = p.kcat / *groups;
  const TileShape& t = TILES[choose_tile(q, 0, EPI_PARTIAL, n_cu, &shared)];
  const long long tiles = (((long long)p.M + t.bm - 1) / t.bm) * (((long long)p.N + t.bn - 1) / t.bn), slots = (long long)t.per_cu * n_cu;
  shared = 1.4 * shared + (double)((tiles + slots - 1) / slots) * bcast_us(t, copies);
  choose_tile(priv, 0, EPI_ROWPAR, n_cu, &us);
  const GemmPair best = best_pair(priv, q, n_cu, copies);
  return pays(1.4 * best.us, shared + 1.4 * us) ? best : pair;
}
hipError_t launch_gemm_shared_private(const GemmPair& pair, int groups, const GemmParams& p, const GemmParams& priv, void* scratch,
                                      hipStream_t s) {
  const hipError_t e = groups == 1 ? launch_any_pair(pair, priv, EPI_ROWPAR, p, EPI_SHARED_BCAST, NormSums{}, s)
                                   : launch_any_pair(pair, priv, EPI_ROWPAR, shared_groups(p, groups, scratch), EPI_PARTIAL, NormSums{}, s);
  return e != hipSuccess || groups == 1 ? e : merge_groups(p, groups, scratch, s);
}

int gemm_route(const GemmParams& p, int layout, int epilogue) {
  GemmParams q = p;
  int groups = 1;
  if (epilogue == EPI_SHARED_BCAST) {
    groups = gemm_shared_groups(p.M, p.N, p.K, p.kcat, gemm_shared_scratch_bytes(p.M, p.N, p.kcat));
    q.G = groups;
    q.kcat = p.kcat / groups;
    if (groups > 1) epilogue = EPI_PARTIAL;
  }
  const int n_cu = compute_units(), route = choose_route(q, layout, epilogue, n_cu);
  if (route != ROUTE_STREAM) return groups > 1 ? 256 * groups + route : route;
  const StreamTile t = choose_stream_tile(q, epilogue, n_cu);
  return t.mt * 16 + t.rt + (t.two_waves ? 128 : 0);
}

}  // namespace caat
