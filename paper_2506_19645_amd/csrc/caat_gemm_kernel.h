// Grouped bf16 shard GEMM kernel template for gfx950 (CDNA4): MFMA 16x16x32 bf16, fp32 accumulation.
//
// One launch covers all T emulated tensor-parallel ranks (group index g).  It implements the two contractions
// of Eq. A3 (column-parallel X_m A_m with the activation fused, row-parallel Y_m B_m with the private-column
// half of the partial channel-reduce + residual fused) and their data / weight gradients.
//
// Tiling: a workgroup owns a BM x BN tile of C and walks K in stages of BKS (64, or 128 where two groups of waves share a
// tile's contraction).  NSTAGE stages of both operand tiles live in LDS and every operand goes global -> LDS directly
// (buffer_load ... lds, no register staging), NSTAGE-1 stages ahead of the MFMAs, so a global / L2 round trip is hidden.
//   * operand contiguous along K in memory (NT's a and b, NN's a): stage = [rows][BKS k], fragment reads are
//     ds_read_b128 (16 consecutive rows x four 16-byte chunks);
//   * operand contiguous along its row index in memory (NN's b, TN's a and b): stage = [BKS k][rows], the memory
//     layout as it is, and the MFMA fragments (8 consecutive k of one row per lane) are gathered by the LDS
//     transpose read ds_read_b64_tr_b16 (16 lanes fetch 4 k-rows x 16 rows and lane j receives row j's 4 k).
// 16-byte chunks are XOR-swizzled (applied on the global side of the copy) so that both kinds of reads are
// bank-conflict free.  Rows / k outside the matrix get an out-of-range buffer offset and arrive as zeros, so
// the main loop has no branch on them.
//
// The accumulator is computed transposed (operands swapped in the MFMA) so that each lane ends up with 4
// consecutive columns of one row of C; the epilogue gathers 8 of them per lane with cross-lane swaps and stores 16
// bytes per lane straight from registers.  With PERSIST a workgroup walks several tiles, whose stages form one stream of
// copies: the first stages of the next tile are in flight while a tile is finished and stored, and the next main loop
// starts without a barrier.  Only half of the waves issue copies (NLOAD below), so that the other half's stores can
// drain under the next tile.  Decode-sized tiles (STREAM_B) may cover fewer output columns than the MFMA tile is wide
// (bn_out).
//
// What bounds the block-sized tiles: the matrix pipes are busy for 49 - 66 % of a launch (waits and barriers of the main loop,
// epilogues that both waves of a SIMD run at the same time), at 1.8 - 1.95 GHz on N(0,1) operands.  A loop of MFMAs on
// registers alone sustains 1.77 PFLOP/s with 32x32x16 and 2.02 with 16x16x32 on such operands, the chip's power limit (2.48 /
// 2.39 on zeros, where both run at full clock), hence the shape.  h = 2048, T = 4, ffn 8192, 8192 tokens, forward GELU /
// row-parallel / GELU' / dX / dA: 263 / 247 / 281 / 243 / 213 us with 32x32x16, an epilogue through LDS and a barrier
// between tiles, 250 / 235 / 271 / 227 / 204 us as it is; 7B SwiGLU (T = 8, 4096 tokens) 670 / 403 / 414 / 608 / 621
// to 626 / 379 / 391 / 557 / 603 us.  Without any epilogue (results dropped) the same launches take 194 / 205 / 220 /
// 203 / 193 us.
#pragma once
#include <type_traits>
#include "caat_internal.h"

namespace caat {

// The lane number as a value the optimiser knows nothing about: what is derived from it inside the tile loop stays there.
// Otherwise per-lane offsets of the copies and of the epilogue are computed once in front of the loop over the tiles
// and, the registers being taken, kept in scratch memory, whose reloads wait for every copy and store in flight.
__device__ __forceinline__ int fresh_lane() {
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  return lane;
}

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef short short8_t __attribute__((ext_vector_type(8)));

static constexpr unsigned OOB = 0x80000000u;  // buffer offset that is always out of range -> load returns 0
static constexpr int DMA_SHIFT = 3072;        // operand windows start this many bytes early (see dma16_group's offsets)

// LDS pointers with a type (address space 3): reads through them are single ds_read instructions with immediate offsets
typedef __attribute__((address_space(3))) const char* lds_c_t;
typedef __attribute__((address_space(3))) const uint4* lds_u4_t;
typedef __attribute__((address_space(3))) short4_t* lds_s4_t;

// rows the LDS image of an operand tile has room for: a power of two (an image [k][rows] is swizzled in whole lines)
constexpr int image_rows(int rows) { return rows == 192 ? 256 : rows; }

template <int BM_, int BN_, int WM_, int WN_, int NSTAGE_ = 2, bool PERSIST_ = true, bool STREAM_B_ = false, int KW_ = 1>
struct TileCfg {
  // KW: groups of waves that share a tile's contraction; group w computes on the w-th 64 k of every stage, and the groups'
  // sums meet in LDS before the epilogue
  static constexpr int KW = KW_;
  static constexpr int BKS = 64 * KW;           // k extent of one LDS stage
  // STREAM_B: decode-sized launches, which read every weight row once (non-temporal copies, bn_out)
  static constexpr bool STREAM_B = STREAM_B_;
  // PERSIST: one workgroup per CU walks several tiles and fetches the next tile's first stages under the epilogue
  static constexpr bool PERSIST = PERSIST_;
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NSTAGE = NSTAGE_;
  static constexpr int NWAVES = WM * WN * KW;
  static constexpr int THREADS = 64 * NWAVES;
  static constexpr int WTM = BM / WM, WTN = BN / WN;  // wave tile
  static constexpr int TM = WTM / 16, TN = WTN / 16;  // 16x16 MFMA tiles per wave
  static constexpr int A_CHUNKS = image_rows(BM) * (BKS / 8);  // uint4 per LDS stage
  static constexpr int STAGE_CHUNKS = A_CHUNKS + image_rows(BN) * (BKS / 8);
  static constexpr int SMEM_CHUNKS = NSTAGE * STAGE_CHUNKS;
  static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be a multiple of 32x32");
  static_assert(!PERSIST || (NSTAGE == 2 && KW == 1), "the persistent loop counts on two slots, and the sums' place is free");
  static_assert((KW - 1) * BM * BN * 4 <= SMEM_CHUNKS * 16, "the groups' sums take the stages' place");
  static_assert(SMEM_CHUNKS * 16 <= 160 * 1024, "LDS capacity");
  // workgroups that fit on one compute unit: LDS (160 KB) and at most 8 waves (2 per SIMD, 256 registers each)
  static constexpr int WGS_PER_CU = ((160 * 1024) / (SMEM_CHUNKS * 16)) < (8 / NWAVES) ? ((160 * 1024) / (SMEM_CHUNKS * 16))
                                                                                        : (8 / NWAVES);
  static constexpr int MIN_WAVES_PER_EU = (NWAVES * WGS_PER_CU) / 4 > 0 ? (NWAVES * WGS_PER_CU) / 4 : 1;
};

// ---- operand contiguous along K: stage [ROWS][BKS k], row = BKS*2 bytes = CPR chunks of 16 bytes; 16 chunks make
// up the 64 LDS banks, so chunk c of row r sits at c ^ swz(r) (128-byte rows: (r>>1)&7, 256-byte rows: r&15):
// 16 consecutive rows then read the same logical chunk from 16 different bank groups.
// One wave instruction fills 64/CPR rows (64 lanes x 16 B, lane order).  `origin` points at the tile's first row;
// rowmap(rr) gives the row of tile row rr RELATIVE to the origin, or -1 if that row does not exist.
template <int ROWS, int NWAVES, int BKS_ = 64, bool GROUPED = true>
struct KContigOperand {
  static constexpr int CPR = BKS_ / 8;           // chunks per row: 8 or 16
  static constexpr int RPI = 64 / CPR;           // rows per copy instruction
  static constexpr int SWZ_SHIFT = CPR == 8 ? 1 : 0;
  static constexpr int NI = ROWS / RPI / NWAVES;  // copy instructions per wave per stage
  // copies that share one LDS base (see dma16_group).  GROUPED: a wave's NI copies fill consecutive 1 KB groups of the
  // stage; otherwise the waves' copies interleave (copy `it` of wave w fills group it*NWAVES + w), which keeps the
  // rows a wave instruction touches in memory next to those of its neighbours: the decode-sized weight streams
  // measured 1-1.5 % faster that way, the block-sized tiles with the grouped issue.
  static constexpr int GRP = !GROUPED ? 1 : (NI % 4 == 0 ? 4 : (NI % 2 == 0 ? 2 : 1));
  static __device__ __forceinline__ int group_of(int wave, int it) { return GROUPED ? wave * NI + it : it * NWAVES + wave; }
  static constexpr int N_VMEM = NI;
  static constexpr int READS_PER_FRAG = 1;
  static_assert(NI % GRP == 0, "whole groups of copies");
  static_assert(CPR == 8 || CPR == 16, "stage depth must be 64 or 128");
  static_assert(ROWS % (RPI * NWAVES) == 0, "rows must divide over the waves");
  static __device__ __forceinline__ int swz(int row) { return (row >> SWZ_SHIFT) & (CPR - 1); }
  const bf16_t* origin;
  unsigned voff[NI];
  int wave;
  int kc[NI];  // logical chunk this lane fetches in copy instruction `it`

  template <class RowMap>
  __device__ __forceinline__ void init(const bf16_t* origin_, long long ld, RowMap rowmap) {
    origin = origin_;
    const int lane = fresh_lane();
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      // a wave's NI copies fill consecutive groups of RPI rows (1 KB of LDS each).  Physical slot lane % CPR of row
      // (wave*NI + it)*RPI + lane / CPR holds logical chunk slot ^ swz(row)
      const int row = group_of(wave, it) * RPI + lane / CPR;
      kc[it] = (lane & (CPR - 1)) ^ swz(row);
      const long long r = rowmap(row);
      // memory-side offsets are relative to a base DMA_SHIFT bytes in front of the operand, less the immediate offset
      // the copy carries as member it % GRP of its group (dma16_group)
      voff[it] = (r >= 0) ? (unsigned)((r * ld + kc[it] * 8) * 2 + DMA_SHIFT - (it % GRP) * 1024) : OOB;
    }
  }
  // koff: element offset of the K-group the stage belongs to (0 unless the contraction runs over several buffers)
  template <bool STREAM = false>
  __device__ __forceinline__ void issue(int k0, int K, uint4* tile, long long koff) const {
    const i32x4_t rs = make_rsrc(reinterpret_cast<const char*>(origin + koff + k0) - DMA_SHIFT);
    if (k0 + BKS_ <= K) {  // a whole stage inside the contraction (all but the last one or two): no per-lane test
#pragma unroll
      for (int gi = 0; gi < NI / GRP; ++gi) dma16_group<STREAM, GRP>(rs, voff + gi * GRP, tile + group_of(wave, gi * GRP) * 64);
      return;
    }
#pragma unroll
    for (int gi = 0; gi < NI / GRP; ++gi) {
      unsigned v[GRP];
#pragma unroll
      for (int j = 0; j < GRP; ++j) v[j] = (k0 + kc[gi * GRP + j] * 8) < K ? voff[gi * GRP + j] : OOB;
      dma16_group<STREAM, GRP>(rs, v, tile + group_of(wave, gi * GRP) * 64);
    }
  }
  // Fragments of a wave whose sub-tile starts at tile row row0 (a multiple of 16): MFMA tile i, k sub-step ks (32 wide):
  // lane (row row0 + 16 i + lane%16, k = 32 ks + 8 (lane/16) ..+7).  The swizzle has a period of 16 rows, so a lane's
  // address is one of two (ks) plus 16 i rows, a constant in the instruction.
  struct Reader {
    lds_c_t p[2];
    // ks0: first of the two 32-wide k sub-steps of the stage that the wave computes on
    __device__ __forceinline__ void init(const uint4* tile, int row0, int ks0, int lane) {
      const int r = lane & 15;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        p[ks] = (lds_c_t)tile + ((row0 + r) * CPR + (((ks0 + ks) * 4 + (lane >> 4)) ^ swz(r))) * 16;
    }
    __device__ __forceinline__ bf16x8_t frag(int stage_bytes, int i, int ks) const {
      return __builtin_bit_cast(bf16x8_t, *(lds_u4_t)(p[ks] + stage_bytes + i * 16 * CPR * 16));
    }
  };
};

// ---- operand contiguous along its row index ([K][rows] in memory): stage [BKS k][ROWS] as in memory, k-row =
// ROWS*2 bytes; chunk c of k-row k sits at c ^ (((k&3)<<2) | (((k>>3)&1)<<1)): the transpose read of 32 lanes (two groups of
// 4 k-rows, 8 apart, 32 bytes of each) then touches every bank once.  With 64 rows two k-rows share a line of all banks, and
// the chunk's swizzle is (((k>>1)&1)<<1) | (((k>>3)&1)<<2).  One wave instruction fills 512/ROWS k-rows.
// `origin` points at (k = 0, first row of the tile); rows_valid = rows of the tile that exist (multiple of 8).
template <int ROWS, int NWAVES, int BKS_ = 64, bool GROUPED = true>
struct RowContigOperand {
  static constexpr int CPR = ROWS / 8;       // chunks per k-row
  static constexpr int KPI = 64 / CPR;       // k-rows per copy instruction
  static constexpr int NI = BKS_ / KPI / NWAVES;
  static constexpr int GRP = !GROUPED ? 1 : (NI % 4 == 0 ? 4 : (NI % 2 == 0 ? 2 : 1));  // as in KContigOperand
  static __device__ __forceinline__ int group_of(int wave, int it) { return GROUPED ? wave * NI + it : it * NWAVES + wave; }
  static constexpr int N_VMEM = NI;
  static constexpr int READS_PER_FRAG = 2;
  static_assert(NI % GRP == 0, "whole groups of copies");
  static_assert((ROWS == 64 || ROWS == 128 || ROWS == 256) && BKS_ % (KPI * NWAVES) == 0, "unsupported tile shape for a transposed operand");
  const bf16_t* origin;
  long long ld;
  unsigned voff[NI];
  int wave, klocal;  // klocal: k-row inside an instruction's group

  template <class RowMap>
  __device__ __forceinline__ void init(const bf16_t* origin_, long long ld_, RowMap rowmap) {
    origin = origin_;
    ld = ld_;
    const int lane = fresh_lane();
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    klocal = lane / CPR;
    const int phys = lane % CPR;
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      const int k = group_of(wave, it) * KPI + klocal;
      const int c = phys ^ swz(k);
      const long long r = rowmap(c * 8);  // 8 consecutive rows share validity (dims % 8 == 0)
      voff[it] = (r >= 0) ? (unsigned)(((long long)k * ld_ + r) * 2 + DMA_SHIFT - (it % GRP) * 1024) : OOB;
    }
  }
  template <bool STREAM = false>
  __device__ __forceinline__ void issue(int k0, int K, uint4* tile, long long koff) const {
    const i32x4_t rs = make_rsrc(reinterpret_cast<const char*>(origin + koff + (long long)k0 * ld) - DMA_SHIFT);
    if (k0 + BKS_ <= K) {  // a whole stage inside the contraction: no per-lane test
#pragma unroll
      for (int gi = 0; gi < NI / GRP; ++gi) dma16_group<STREAM, GRP>(rs, voff + gi * GRP, tile + group_of(wave, gi * GRP) * 64);
      return;
    }
#pragma unroll
    for (int gi = 0; gi < NI / GRP; ++gi) {
      unsigned v[GRP];
#pragma unroll
      for (int j = 0; j < GRP; ++j) {
        const int k = group_of(wave, gi * GRP + j) * KPI + klocal;
        v[j] = (k0 + k < K) ? voff[gi * GRP + j] : OOB;
      }
      dma16_group<STREAM, GRP>(rs, v, tile + group_of(wave, gi * GRP) * 64);
    }
  }
  static __device__ __forceinline__ int swz(int k) {
    return ROWS == 64 ? (((k >> 1) & 1) << 1) | (((k >> 3) & 1) << 2) : ((k & 3) << 2) | (((k >> 3) & 1) << 1);
  }
  // The same fragments as KContigOperand::Reader, each gathered by two transpose reads of 4 k.  A lane fetches 8 bytes
  // (rows 4 (lane%4) ..+3 of the 16) of k-row 32 ks + 8 (lane/16) + (lane%16)/4 and of the k-row 4 further on; both have
  // the same swizzle.  TT = MFMA tiles of the wave: the tile index moves the chunk inside the swizzle, so there is an
  // address per tile (up to eight: 8 tiles are one swizzle period); ks is a constant in the instruction.
  struct Reader {
    lds_c_t p[8];
    __device__ __forceinline__ void init(const uint4* tile, int row0, int ks0, int lane) {
      const int i16 = lane & 15, k = (lane >> 4) * 8 + (i16 >> 2);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int m = row0 + i * 16 + (i16 & 3) * 4;
        p[i] = (lds_c_t)tile + (ks0 * 32 + k) * (ROWS * 2) + ((((m >> 3) ^ swz(k)) << 4) + ((m & 7) << 1));
      }
    }
    __device__ __forceinline__ bf16x8_t frag(int stage_bytes, int i, int ks) const {
      const lds_c_t q = p[i] + stage_bytes + ks * 32 * (ROWS * 2);
      const short4_t v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_t)q);
      const short4_t v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_t)(q + 4 * (ROWS * 2)));
      const short8_t v = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
      return __builtin_bit_cast(bf16x8_t, v);
    }
  };
};

template <bool ROWCONTIG, int ROWS, int NWAVES, int BKS_, bool GROUPED>
struct OperandSel { typedef KContigOperand<ROWS, NWAVES, BKS_, GROUPED> type; };
template <int ROWS, int NWAVES, int BKS_, bool GROUPED>
struct OperandSel<true, ROWS, NWAVES, BKS_, GROUPED> { typedef RowContigOperand<image_rows(ROWS), NWAVES, BKS_, GROUPED> type; };

// Which weight row (relative to the tile's first row n0) lies in row rr of the B tile in LDS, or -1 for none.  Plain
// epilogues: rows in order, as many as the tile covers (bn_out) and the matrix has.  SwiGLU: each wave's WTN tile rows
// are 32 gate rows, then the 32 up rows of the same output columns (`half` rows further down), and so on, so that an
// accumulator pair of a wave holds gate and up of the same 32 outputs.  RoPE: a wave's 64 tile rows are channels j .. j + 31 of a
// head of 128 and the 32 that they are rotated with, 64 further on.
template <class CFG, bool SWI, bool ROPE>
__device__ __forceinline__ long long b_tile_row(int rr, int n0, int bn_out, int N, int half) {
  if constexpr (SWI) {
    const int w = rr / CFG::WTN, rw = rr - w * CFG::WTN;
    const int j = rw >> 5, c = rw & 31;
    const int col = (w * (CFG::WTN / 64) + (j >> 1)) * 32 + c;  // output column relative to n0
    if (col >= bn_out || n0 + col >= half) return -1;
    return (long long)col + ((j & 1) ? half : 0);
  } else if constexpr (ROPE) {
    const int w = rr >> 6, col = (w >> 1) * 128 + (w & 1) * 32 + (rr & 32) * 2 + (rr & 31);
    return n0 + col < N ? (long long)col : -1;
  } else {
    const int nrem = (N - n0) < bn_out ? (N - n0) : bn_out;
    return rr < nrem ? (long long)rr : -1;
  }
}

// The tiles of workgroup `bid` of `nb` that share a launch (nb a multiple of 8, or bid is blockIdx.x: bid % 8 names the XCD).
template <class CFG, bool AT, bool BT, int EPI>
__device__ __forceinline__ void gemm_tiles(const GemmParams& p, uint4* smem, int bid, int nb) {
  constexpr int BM = CFG::BM, BN = CFG::BN, NSTAGE = CFG::NSTAGE;
  constexpr int TM = CFG::TM, TN = CFG::TN, WTM = CFG::WTM, WTN = CFG::WTN;
  constexpr bool SWI = (EPI == EPI_SWIGLU_FWD);
  constexpr int BN_OUT = SWI ? BN / 2 : BN;  // output columns covered by one tile
  static_assert(!SWI || WTN % 64 == 0, "SwiGLU pairing needs 32 gate and 32 up columns per wave");
  constexpr bool ROPE = (EPI == EPI_ROPE);
  static_assert(!ROPE || (WTN == 64 && BN % 128 == 0), "a wave rotates 32 channels of a head with the 32 that lie 64 further on");

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = CFG::KW > 1 ? wave / (CFG::WM * CFG::WN) : 0;   // group of waves (KW)
  const int wt = wave - kw * (CFG::WM * CFG::WN);                // wave of the group
  const int wm = wt / CFG::WN;
  const int wn = wt - wm * CFG::WN;

  // ---- tiles of this workgroup.  Tile ids are cut into 8 contiguous ranges, one per XCD (workgroup b runs on XCD
  // b % 8), so that the workgroups sharing an L2 work on neighbouring tiles; inside a range the workgroups of the XCD
  // take tiles round-robin.  A tile id maps to (rank g, tile row, tile column) in a grouped (8 tile rows) order.
  // Decode-sized tiles may be told to cover fewer output columns than the MFMA tile is wide (bn_out, a multiple of
  // 8): the kernel is then a weight stream, and what counts is that every compute unit gets the same number of weight
  // rows.  The rows beyond bn_out are not fetched (out-of-range copy offsets) and their columns are not stored.
  constexpr bool NARROW = CFG::STREAM_B;
  const int bn_out = (NARROW && p.bn_out > 0) ? p.bn_out : BN_OUT;
  const int tiles_m = (p.M + BM - 1) / BM;
  const int tiles_n = (p.N + bn_out - 1) / bn_out;
  const int tiles = tiles_m * tiles_n;
  const int total = tiles * p.G;
  int pid, pid_end, pid_step;
  {
    const int q = total >> 3, rem = total & 7, x = bid & 7;
    const int start = x * q + (x < rem ? x : rem);
    pid_end = start + q + (x < rem ? 1 : 0);
    pid = start + (bid >> 3);
    pid_step = (nb - x + 7) >> 3;  // workgroups on this XCD
  }

  constexpr int BKS = CFG::BKS;         // this instantiation's stage depth (hides the namespace default)
  constexpr int NSUB = 2;               // 32-wide k sub-steps (one MFMA deep) of a wave per stage
  // Waves that issue the global -> LDS copies.  A wave's copies and its epilogue stores complete in issue order on one
  // counter, so a wave that copies has to let its stores drain before it can wait for the next tile's second stage,
  // and the stores of all compute units come as one chip-wide burst (the workgroups run in lockstep) that takes
  // several k steps when a tile has several outputs.  In the persistent eight-wave tiles only the first four waves
  // copy (twice the instructions each, one such wave per SIMD next to a wave that only computes): the other four never
  // wait on that counter in the main loop, and their half of the stores drains under the next tile.  Measured: forward
  // SwiGLU GEMM -5 %, GELU' GEMM -5 %, weight gradients -2.4 %, QKV -3 %; nothing lost anywhere.
  constexpr int NLOAD = (CFG::PERSIST && CFG::NWAVES == 8) ? 4 : CFG::NWAVES;
  const bool loader = wave < NLOAD;
  typedef typename OperandSel<AT, BM, NLOAD, BKS, !CFG::STREAM_B>::type OpA;
  typedef typename OperandSel<BT, BN, NLOAD, BKS, !CFG::STREAM_B>::type OpB;
  OpA la;
  OpB lb;
  // rank g, first row m0 and first column n0 of a tile
  auto tile_coords = [&](int id, int& g, int& m0, int& n0) {
    g = id / tiles;
    const int t = id - g * tiles;
    constexpr int GROUP = 8;
    const int width = GROUP * tiles_n;
    const int grp = t / width;
    const int first = grp * GROUP;
    const int gsize = (tiles_m - first) < GROUP ? (tiles_m - first) : GROUP;
    const int r = t - grp * width;
    m0 = (first + r % gsize) * BM;
    n0 = (r / gsize) * bn_out;
  };
  auto setup_copies = [&](int id) {   // la, lb onto tile id
    int g, m0, n0;
    tile_coords(id, g, m0, n0);
    const bf16_t* ag = p.a + (long long)g * p.stride_a;
    const bf16_t* bg = p.b + (long long)g * p.stride_b;
    const int mrem = p.M - m0 < BM ? p.M - m0 : BM;   // an image may have room for more rows than the tile has
    la.init(AT ? ag + m0 : ag + (long long)m0 * p.lda, p.lda,
            [=](int rr) -> long long { return (rr < mrem) ? (long long)rr : -1; });
    if constexpr (!BT) {
      const int n0c = n0, bnc = bn_out, Nc = p.N, halfc = p.half;
      auto rowmap = [=](int rr) -> long long { return b_tile_row<CFG, SWI, ROPE>(rr, n0c, bnc, Nc, halfc); };
      lb.init(bg + (long long)n0 * p.ldb, p.ldb, rowmap);
    } else {
      const int nrem = p.N - n0 < BN ? p.N - n0 : BN;
      lb.init(bg + n0, p.ldb, [=](int rr) -> long long { return (rr < nrem) ? (long long)rr : -1; });
    }
  };

  // With the broadcast and the partial-sum epilogue the contraction index runs over kcat buffers of K each (operand g' of both a and b lies
  // kstride elements after operand g'-1): that is how the sum over ranks of Eq. A3's shared channels is taken inside
  // the accumulator.  Every other instantiation keeps the single-buffer code (no per-stage bookkeeping).
  constexpr bool KCAT = (EPI == EPI_SHARED_BCAST || EPI == EPI_PARTIAL);
  const int K = p.K;
  const int kcat = KCAT ? (p.kcat > 1 ? p.kcat : 1) : 1;
  const int nkg = (K + BKS - 1) / BKS;   // stages of one K-group
  const int nk = nkg * kcat;             // stages of a tile
  constexpr int A_CHUNKS = CFG::A_CHUNKS;
  constexpr int STAGE_BYTES = CFG::STAGE_CHUNKS * 16;
  constexpr int NV = OpA::N_VMEM + OpB::N_VMEM;  // copies of a loading wave per stage
  // decode-sized launches (at most 64 token rows per rank: one tile row) read every weight row exactly once
  constexpr bool B_STREAM = CFG::STREAM_B;

  // ---- the loading side.  The stages of all tiles of this workgroup form one stream; issue_one copies the next one
  // into the next slot, and steps on to the next tile behind a tile's last stage: the first stages of a tile are on
  // their way while the tile before is still computed and stored.
  int lpid = pid;          // tile of the next copy
  int lstage = 0;          // its stage (inside its K-group)
  int lkg = 0;             // its K-group
  int lslot = 0;           // slot it goes to
  bool lmore = pid < pid_end;
  auto issue_one = [&]() {
    if (!lmore) return;
    if (loader) {
      uint4* slot = smem + lslot * CFG::STAGE_CHUNKS;
      if constexpr (KCAT) {
        la.issue(lstage * BKS, K, slot, (long long)lkg * p.kstride_a);
        lb.template issue<B_STREAM>(lstage * BKS, K, slot + A_CHUNKS, (long long)lkg * p.kstride_b);
      } else {
        la.issue(lstage * BKS, K, slot, 0);
        lb.template issue<B_STREAM>(lstage * BKS, K, slot + A_CHUNKS, 0);
      }
    }
    lslot = lslot + 1 == NSTAGE ? 0 : lslot + 1;
    if (++lstage == nkg) {
      lstage = 0;
      if (KCAT && ++lkg < kcat) return;
      lkg = 0;
      lpid += pid_step;
      lmore = CFG::PERSIST && lpid < pid_end;
      if (lmore && loader) setup_copies(lpid);
    }
  };

  constexpr int TMH = TM / 2;                    // MFMA tile rows of half a wave tile
  static_assert(TM % 2 == 0 && NSUB % 2 == 0, "the main loop takes a wave's tile rows in two halves, two sets of columns");
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
  typename OpA::Reader ra;
  typename OpB::Reader rb;
  ra.init(smem, wm * WTM, kw * NSUB, lane);
  rb.init(smem + A_CHUNKS, wn * WTN, kw * NSUB, lane);

  constexpr int NS = WTN / 32;                   // 32-column groups of a wave's sub-tile
  // epilogue stores per wave and tile (known at compile time except for the broadcast epilogue's loop over ranks; RoPE's
  // stores to the caches are not counted: the wait that counts on this number waits for some of them too)
  constexpr int EPI_STORES =
      (EPI == EPI_SHARED_BCAST)
          ? 1000
          : EPI == EPI_PARTIAL ? TM * TN : TM * (SWI ? NS / 2 : NS) * (EPI == EPI_SWIGLU_FWD ? 3 : ((EPI == EPI_GELU_FWD || EPI == EPI_SWIGLU_BWD) ? 2 : 1));

  if (pid >= pid_end) return;
  if (loader) setup_copies(pid);
#pragma unroll
  for (int q = 0; q < NSTAGE; ++q) issue_one();
  // copies complete in order: with at most the NSTAGE-1 newer stages outstanding, the first one has landed
  if (loader) {
    if (lmore) wait_vmcnt<(NSTAGE - 1) * NV>();
    else wait_vmcnt<0>();
  }
  __syncthreads();
  int cur = 0;                       // LDS offset of the stage being computed
  bool behind_stores = false;        // this wave's stores of the tile before stand behind this tile's second stage

  while (true) {
    f32x4_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;

    // ---- main loop.  A wave's MFMAs of a k sub-step run in two halves of its tile rows: half 0 computes on aq[0] while
    // the fragments of half 1 are read into aq[1], half 1 computes on aq[1] while aq[0] and the other set of bq are
    // filled for the next sub-step.  In the last sub-step of a stage nothing of the stage is left to read after half 0:
    // there all waves meet, the next stage has landed, and the next copies go into the slot just freed (one barrier per
    // stage, NSTAGE-1 whole stages of lead for a copy).  One MFMA per step with its share of the reads right behind it:
    // a wave issues in order, and the fences keep the steps in order.  The columns are taken to and fro, so that one operand
    // of an MFMA is that of the MFMA before: on N(0,1) operands, where the chip's power sets the clock, MFMAs on registers
    // alone sustain 2.10 PFLOP/s in this order, 2.05 with every row from its first column on and 1.99 with both operands new
    // each time; the GEMM of 4 x 8192 x 2048 x 2048 goes from 209 / 216 to 206 / 212 us (NT / NN).
    bf16x8_t aq[2][TMH], bq[2][TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bq[0][j] = rb.frag(cur, j, 0);
#pragma unroll
    for (int i = 0; i < TMH; ++i) aq[0][i] = ra.frag(cur, i, 0);
    fence();
    auto stage = [&](int kt, auto last_c) {
      constexpr bool LAST = decltype(last_c)::value;
      const int nxt = cur + STAGE_BYTES == NSTAGE * STAGE_BYTES ? 0 : cur + STAGE_BYTES;
#pragma unroll
      for (int ss = 0; ss < NSUB; ++ss) {
        constexpr int NM = TMH * TN;
        const bool tail = ss + 1 == NSUB;
#pragma unroll
        for (int m = 0; m < NM; ++m) {   // half 0; reads: half 1's rows of the same sub-step
          const int i = m / TN, j = i & 1 ? TN - 1 - m % TN : m % TN;
          // operands swapped: the accumulator holds C^T, i.e. lane = row of C, registers = columns of C
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bq[ss & 1][j], aq[0][i], acc[i][j], 0, 0, 0);
#pragma unroll
          for (int r = m * TMH / NM; r < (m + 1) * TMH / NM; ++r) aq[1][r] = ra.frag(cur, TMH + r, ss);
          fence();
        }
        if (tail) {
          if (loader) {
            // the next stage has landed: newer are NSTAGE-2 stages and, in a tile's first stage, the stores of the tile
            // before (a fixed number, issued after this tile's second stage), which may stay in flight
            if (EPI_STORES <= 63 && behind_stores) wait_vmcnt<EPI_STORES <= 63 ? EPI_STORES : 0>();
            else if (lmore) wait_vmcnt<(NSTAGE - 2) * NV>();
            else wait_vmcnt<0>();
            behind_stores = false;
          }
          __syncthreads();
          fence();
          issue_one();
        }
#pragma unroll
        for (int m = 0; m < NM; ++m) {   // half 1; reads: half 0's rows and all columns of the next sub-step
          const int i = m / TN, j = i & 1 ? TN - 1 - m % TN : m % TN;
          acc[TMH + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bq[ss & 1][j], aq[1][i], acc[TMH + i][j], 0, 0, 0);
          if (!(LAST && tail)) {
            constexpr int NR = TMH + TN;
#pragma unroll
            for (int r = m * NR / NM; r < (m + 1) * NR / NM; ++r) {
              if (r < TN) bq[(ss + 1) & 1][r] = rb.frag(tail ? nxt : cur, r, tail ? 0 : ss + 1);
              else aq[0][r - TN] = ra.frag(tail ? nxt : cur, r - TN, tail ? 0 : ss + 1);
            }
          }
          fence();
        }
      }
      cur = nxt;
    };
#pragma clang loop unroll(disable)
    for (int kt = 0; kt + 1 < nk; ++kt) stage(kt, std::false_type{});
    stage(nk - 1, std::true_type{});

    if constexpr (CFG::KW > 1) {
      // The sums of the groups meet in LDS (no copy is in flight and nothing is read from the stages any more once all
      // waves are here), in ascending order; group 0 goes on to the epilogue.
      __syncthreads();
      f32x4_t* part = reinterpret_cast<f32x4_t*>(smem) + wt * (TM * TN * 64) + lane;
      constexpr int GROUP_VECS = CFG::WM * CFG::WN * TM * TN * 64;
      if (kw > 0) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) part[(kw - 1) * GROUP_VECS + (i * TN + j) * 64] = acc[i][j];
      }
      __syncthreads();
      if (kw > 0) return;
#pragma unroll
      for (int w = 1; w < CFG::KW; ++w)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] += part[(w - 1) * GROUP_VECS + (i * TN + j) * 64];
    }

    // ---- epilogue.  Each lane holds C[row = lane%16][col = 4*(lane/16) + 0..3] of every 16x16 tile.  Stored as they
    // are, these 8-byte pieces would leave as 32-byte runs; so two neighbouring tiles exchange pieces between the
    // 16-lane groups (v_permlane16_swap: odd groups of the first against even groups of the second), after which a lane
    // holds 8 consecutive columns of its row and the four lanes of a row 64 contiguous bytes, without a trip through
    // LDS.  Where the wave has 64 output columns, lanes 8 apart exchange once more (DPP rotation by 8): an instruction
    // then writes whole 128-byte lines of 8 rows (half lines with the non-temporal hint cost the data-gradient GEMM of
    // the 7B shape 5 %: 590 against 559 us).  The fused element-wise work (activation, its derivative, the private half of the partial channel-reduce +
    // residual) happens on these vectors.
    //
    // Every global access of the epilogue is a raw buffer load / store whose offset is replaced by an out-of-range
    // one where the row or column does not exist (the load then returns zero, the store is dropped): the code has no
    // branch, so the number of vector-memory instructions per tile is fixed (the wait in the next tile's first stage
    // counts on it) and the compiler's own waits for the prefetched second operand stay exact.
    int eg, em0, en0;
    tile_coords(pid, eg, em0, en0);
    const int elane = fresh_lane();
    const int eq = elane >> 4;
    const int ecol0 = (eq & 1) * 16 + (eq >> 1) * 8;   // the lane's 8 columns of a 32-column group
    auto unpack = [](const uint4& v, float* f) {
      f[0] = lo_bf(v.x); f[1] = hi_bf(v.x); f[2] = lo_bf(v.y); f[3] = hi_bf(v.y);
      f[4] = lo_bf(v.z); f[5] = hi_bf(v.z); f[6] = lo_bf(v.w); f[7] = hi_bf(v.w);
    };
    auto pack = [](const float* f) -> uint4 {
      return make_uint4(pack2bf(f[0], f[1]), pack2bf(f[2], f[3]), pack2bf(f[4], f[5]), pack2bf(f[6], f[7]));
    };
    // the lane's 8 columns of 32-column group s, row 16 i + lane%16, rounded to bf16
    auto rounded = [&](int i, int s) -> uint4 {
      const f32x4_t x = acc[i][2 * s], y = acc[i][2 * s + 1];
      const auto lo = __builtin_amdgcn_permlane16_swap(pack2bf(x[0], x[1]), pack2bf(y[0], y[1]), false, false);
      const auto hi = __builtin_amdgcn_permlane16_swap(pack2bf(x[2], x[3]), pack2bf(y[2], y[3]), false, false);
      return make_uint4(lo[0], hi[0], lo[1], hi[1]);
    };
    // Output vectors per lane and 16 rows (SwiGLU: group 2s gate, 2s+1 up).  LINES: two vectors, whole lines of 8 rows
    // each: vector v belongs to row 16 i + 8 v + lane%8 and to column group (lane/8)%2.
    constexpr int NO = SWI ? NS / 2 : NS;
    constexpr bool LINES = !SWI && NS == 2;
    auto vectors = [&](int i, uint4* v) {
#pragma unroll
      for (int st = 0; st < NO; ++st) v[st] = rounded(i, st);
      if constexpr (LINES) {
        auto swap8 = [](unsigned& a, unsigned& b) {   // lanes 8-15 of a against lanes 0-7 of b, in every 16 lanes
          const unsigned a0 = a, b0 = b;
          a = (unsigned)__builtin_amdgcn_update_dpp((int)a0, (int)b0, 0x128, 0xF, 0xC, false);
          b = (unsigned)__builtin_amdgcn_update_dpp((int)b0, (int)a0, 0x128, 0xF, 0x3, false);
        };
        swap8(v[0].x, v[1].x);
        swap8(v[0].y, v[1].y);
        swap8(v[0].z, v[1].z);
        swap8(v[0].w, v[1].w);
      }
    };
    constexpr bool HAS_AUX = (EPI == EPI_ROWPAR || EPI == EPI_GELU_BWD || EPI == EPI_SWIGLU_BWD);
    constexpr int AUXV = (EPI == EPI_SWIGLU_BWD) ? 2 : 1;
    const int wrow0 = em0 + wm * WTM;             // first row of the wave's sub-tile
    const int wcol0 = en0 + wn * (SWI ? WTN / 2 : WTN);  // first output column of the wave's sub-tile
    const int ncols = SWI ? p.half : p.N;
    // buffer windows start at the wave's first row, so that offsets stay small: row in the sub-tile * ld + column, in bytes
    const rsrc_t rc = make_rsrc_t(p.c + (long long)eg * p.stride_c + (long long)wrow0 * p.ldc);
    const rsrc_t rc2 = make_rsrc_t((EPI == EPI_GELU_FWD || SWI) ? p.c2 + (long long)eg * p.stride_c2 + (long long)wrow0 * p.ldc2 : p.c);
    const rsrc_t raux = make_rsrc_t(HAS_AUX ? p.aux + (long long)eg * p.stride_aux + (long long)wrow0 * p.ldaux : p.c);
    int erow[NO], ecol[NO];                       // row (of 16) and first output column of the lane's vector st
    unsigned voff_c[NO], voff_c2[NO], voff_aux[NO];
#pragma unroll
    for (int st = 0; st < NO; ++st) {
      erow[st] = LINES ? (elane & 7) + 8 * st : elane & 15;
      ecol[st] = wcol0 + (LINES ? (elane >> 3) & 1 : st) * 32 + ecol0;
      const bool colok = ecol[st] < ncols && ecol[st] - en0 < bn_out;
      voff_c[st] = colok ? (unsigned)((erow[st] * p.ldc + ecol[st]) * 2) : OOB;
      voff_c2[st] = colok ? (unsigned)((erow[st] * p.ldc2 + ecol[st]) * 2) : OOB;
      // the residual is only needed where the vector has a private channel (Eq. A3)
      const bool auxok = colok && (EPI != EPI_ROWPAR || ecol[st] + 7 >= p.hs);
      voff_aux[st] = auxok ? (unsigned)((erow[st] * p.ldaux + ecol[st]) * 2) : OOB;
    }
    auto row_ok = [&](int i, int st) { return i * 16 + erow[st] < p.M - wrow0; };
    // epilogues that read a second tensor (residual, saved pre-activations) fetch it AUXD 16-row slabs ahead: a slab's
    // conversion and stores take less time than one trip to memory.  The residual epilogue, light on registers, fetches
    // all of the wave's slabs at once.
    constexpr int AUXD = !HAS_AUX ? 1 : (EPI == EPI_ROWPAR ? TM : (TM < 4 ? TM : 4));
    u32x4_t auxbuf[AUXD][HAS_AUX ? NO * AUXV : 1];
    auto aux_fetch = [&](int i, u32x4_t* buf) {
      const int so = i * 16 * (int)p.ldaux * 2;
#pragma unroll
      for (int st = 0; st < NO; ++st) {
        const unsigned vo = row_ok(i, st) ? voff_aux[st] : OOB;
        // read once by this tile only: non-temporal hint (cache policy bit 1)
        buf[st * AUXV] = __builtin_amdgcn_raw_buffer_load_b128(raux, vo, so, 2);
        if constexpr (AUXV == 2) buf[st * AUXV + 1] = __builtin_amdgcn_raw_buffer_load_b128(raux, vo, so + p.half * 2, 2);
      }
    };
    auto to_u4 = [](const u32x4_t& v) -> uint4 { return make_uint4(v[0], v[1], v[2], v[3]); };
    // Stores keep the slab offset in the vector offset and pass no scalar offset register: the 16-byte store reads
    // its data registers a few cycles after it issues, and the compiler only keeps the following instructions from
    // overwriting them (the documented store-data hazard) for the form without a scalar offset register; with one,
    // the first data register was now and then overwritten by the next vector's arithmetic before the store had
    // read it (seen as a wrong first dword in a few lanes at full problem sizes).  The two idle cycles after the
    // store restate that requirement where the store is issued.
    auto put = [&](const rsrc_t& r, const uint4& v, bool ok, unsigned vo, int so) {
      const u32x4_t w = {v.x, v.y, v.z, v.w};
      __builtin_amdgcn_raw_buffer_store_b128(w, r, ok ? vo + (unsigned)so : OOB, 0, 0);
      asm volatile("s_nop 1" ::: "memory");
    };
    // the same for a tensor that nothing reads before the backward pass (saved pre-activations): non-temporal hint,
    // so that it does not push the activation the next GEMM is about to read out of the caches
    auto put_late = [&](const rsrc_t& r, const uint4& v, bool ok, unsigned vo, int so) {
      const u32x4_t w = {v.x, v.y, v.z, v.w};
      __builtin_amdgcn_raw_buffer_store_b128(w, r, ok ? vo + (unsigned)so : OOB, 0, 2);
      asm volatile("s_nop 1" ::: "memory");
    };
    // The slab loop exists three times for the row-parallel epilogue: a tile that lies entirely left of hs holds
    // shared channels only (Eq. A3: every rank's partial sum goes out as it is, the reduce adds the residual), so it
    // needs neither the residual fetch nor the case split and runs the plain store path; a tile entirely right of hs
    // needs no case split; only a tile that contains hs takes the general code.  All versions issue the same number
    // of stores, and each is free of branches in itself.
    auto slabs = [&](auto tile_kind) {
      constexpr bool SH = decltype(tile_kind)::value == 1;    // shared channels only
      constexpr bool PRIV = decltype(tile_kind)::value == 2;  // private channels only
      if constexpr (HAS_AUX && !SH) {
#pragma unroll
        for (int i = 0; i < AUXD && i < TM; ++i) aux_fetch(i, auxbuf[i]);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        uint4 vec[NS];
        if constexpr (SWI) {
#pragma unroll
          for (int q = 0; q < NS; ++q) vec[q] = rounded(i, q);
        } else {
          vectors(i, vec);
        }
        const int so_c = i * 16 * (int)p.ldc * 2, so_c2 = i * 16 * (int)p.ldc2 * 2;
#pragma unroll
        for (int st = 0; st < NO; ++st) {
          const bool rowok = row_ok(i, st);
          const unsigned vo = voff_c[st];
          if constexpr (SWI) {
            const uint4 gw = vec[2 * st], uw = vec[2 * st + 1];
            float gt[8], up[8], y[8];
            unpack(gw, gt);
            unpack(uw, up);
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = gt[e] * sigmoid_f(gt[e]) * up[e];
            put_late(rc, gw, rowok, vo, so_c);
            put_late(rc, uw, rowok, vo, so_c + p.half * 2);
            put(rc2, pack(y), rowok, voff_c2[st], so_c2);
          } else {
            const uint4 raw = vec[st];
            if constexpr (EPI == EPI_PLAIN) {
              if (p.late_c) put_late(rc, raw, rowok, vo, so_c);
              else put(rc, raw, rowok, vo, so_c);
            } else if constexpr (EPI == EPI_GELU_FWD) {
              // the activation is taken of the bf16-rounded pre-activation, the value the backward pass sees too
              float v[8], y[8];
              unpack(raw, v);
#pragma unroll
              for (int e = 0; e < 8; ++e) y[e] = gelu_f(v[e]);
              put_late(rc, raw, rowok, vo, so_c);
              put(rc2, pack(y), rowok, voff_c2[st], so_c2);
            } else if constexpr (EPI == EPI_ROWPAR && SH) {
              put(rc, raw, rowok, vo, so_c);  // a tile of shared channels only: this rank's partial sums as they are
            } else if constexpr (EPI == EPI_ROWPAR) {
              // Eq. A3 case split, private side: columns >= hs are final here (scale, + residual); columns < hs are
              // stored as this rank's partial sum for the reduce kernel (rounding a bf16 value to bf16 again leaves
              // its bits as they are).  The private value is scaled from the bf16-rounded partial.
              float v[8], r[8];
              unpack(raw, v);
              unpack(to_u4(auxbuf[i % AUXD][st]), r);
#pragma unroll
              for (int e = 0; e < 8; ++e) v[e] = (PRIV || ecol[st] + e >= p.hs) ? p.scale * v[e] + r[e] : v[e];
              put(rc, pack(v), rowok, vo, so_c);
            } else if constexpr (EPI == EPI_SHARED_BCAST) {
              // Eq. A3, shared channels with the sum over ranks already in the accumulator: every rank's output gets
              // the same sum plus that rank's residual
              float v[8];
              unpack(raw, v);
              for (int m = 0; m < p.bcast; ++m) {
                const rsrc_t rr = make_rsrc_t(p.aux + (long long)m * p.stride_aux + (long long)wrow0 * p.ldaux);
                const rsrc_t rw = make_rsrc_t(p.c + (long long)m * p.stride_c + (long long)wrow0 * p.ldc);
                const unsigned va = rowok ? voff_aux[st] : OOB;
                float r[8], o[8];
                unpack(to_u4(__builtin_amdgcn_raw_buffer_load_b128(rr, va, i * 16 * (int)p.ldaux * 2, 0)), r);
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = v[e] + r[e];
                put(rw, pack(o), rowok, vo, so_c);
              }
            } else if constexpr (EPI == EPI_GELU_BWD) {
              float v[8], pr[8];
              unpack(raw, v);
              unpack(to_u4(auxbuf[i % AUXD][st]), pr);
#pragma unroll
              for (int e = 0; e < 8; ++e) v[e] *= gelu_grad_f(pr[e]);
              put(rc, pack(v), rowok, vo, so_c);
            } else if constexpr (EPI == EPI_SWIGLU_BWD) {
              float v[8], gt[8], up[8], dg[8], du[8];
              unpack(raw, v);
              unpack(to_u4(auxbuf[i % AUXD][st * AUXV]), gt);
              unpack(to_u4(auxbuf[i % AUXD][st * AUXV + (AUXV - 1)]), up);
#pragma unroll
              for (int e = 0; e < 8; ++e) {
                const float sg = sigmoid_f(gt[e]);
                dg[e] = v[e] * up[e] * sg * (1.0f + gt[e] * (1.0f - sg));
                du[e] = v[e] * gt[e] * sg;
              }
              put(rc, pack(dg), rowok, vo, so_c);
              put(rc, pack(du), rowok, vo, so_c + p.half * 2);
            }
          }
        }
        if constexpr (HAS_AUX && !SH) {
          if (i + AUXD < TM) aux_fetch(i + AUXD, auxbuf[i % AUXD]);  // this slab's registers are free again
        }
      }
    };
    if constexpr (EPI == EPI_PARTIAL) {
      // fp32 sums as they are: 16 bytes per lane, 64 contiguous bytes per row and MFMA tile.  The merge reads them next.
      float* cf = reinterpret_cast<float*>(p.c) + (long long)eg * p.stride_c + (long long)wrow0 * p.ldc;
      const rsrc_t rf = make_rsrc_t(cf);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = i * 16 + (elane & 15);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int col = wcol0 + j * 16 + 4 * eq;
          const bool ok = row < p.M - wrow0 && col < ncols && col - en0 < bn_out;
          const uint4 w = __builtin_bit_cast(uint4, acc[i][j]);
          put(rf, w, ok, (unsigned)((row * p.ldc + col) * 4), 0);
        }
      }
    } else if constexpr (ROPE) {
      // q and k are rotated as they were rounded, 8 pairs (j, j + 64) of a row per lane.  A sine and a cosine for each pair and
      // row would cost more than the pass over q and k that this saves: 16 rows on the angle has grown by the same amount for
      // every lane, so the pair is turned by that (fp32; 8 steps at most, 1e-6 against the 1e-4 of an fp32 frequency), and it
      // is only taken anew where the sequence ended in between.
      const int head = en0 + (wn >> 1) * 128;          // first column of the wave's head
      const int j0 = (wn & 1) * 32 + ecol0;            // the lane's first pair
      const bool rot = head < p.rope.q + p.rope.k;
      const unsigned seq = (unsigned)p.rope.seq;
      const unsigned vo = head < p.N ? (unsigned)(((elane & 15) * p.ldc + head + j0) * 2) : OOB;
      bf16_t* cache = nullptr;
      if (p.rope.kc && head >= p.rope.q && head < p.N) cache = rot ? p.rope.kc : p.rope.vc;
      const int kv = (head - p.rope.q) / 128 - (rot ? 0 : p.rope.k / 128);
      float sn[8] = {}, cs[8] = {}, sn16[8] = {}, cs16[8] = {};
      int until = 0;                                   // rows from wrow0 on that lie in the sequence of the row before
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = i * 16 + (elane & 15);
        const bool rowok = row < p.M - wrow0;
        uint4 lo = rounded(i, 0), hi = rounded(i, 1);
        if (rot) {
          if (16 * i + 15 < until) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float c = cs[e] * cs16[e] - sn[e] * sn16[e];
              sn[e] = sn[e] * cs16[e] + cs[e] * sn16[e];
              cs[e] = c;
            }
          } else {
            until = 16 * i + (int)(seq - (unsigned)(wrow0 + 16 * i) % seq);
            const float pos = (float)((unsigned)(wrow0 + row) % seq);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float2 f = rope_freq(j0 + e, 128, p.rope.log2_base);
              rope_sincos(pos, f, sn[e], cs[e]);
              rope_sincos(16.0f, f, sn16[e], cs16[e]);
            }
          }
          auto turn = [&](unsigned& a, unsigned& b, int e) {
            const float x0 = lo_bf(a), x1 = hi_bf(a), y0 = lo_bf(b), y1 = hi_bf(b);
            a = pack2bf(x0 * cs[e] - y0 * sn[e], x1 * cs[e + 1] - y1 * sn[e + 1]);
            b = pack2bf(y0 * cs[e] + x0 * sn[e], y1 * cs[e + 1] + x1 * sn[e + 1]);
          };
          turn(lo.x, hi.x, 0);
          turn(lo.y, hi.y, 2);
          turn(lo.z, hi.z, 4);
          turn(lo.w, hi.w, 6);
        }
        const int so = i * 16 * (int)p.ldc * 2;
        put(rc, lo, rowok, vo, so);
        put(rc, hi, rowok && vo != OOB, vo + 128, so);
        if (cache && rowok) {
          // the caches are read by later decode steps, not by this layer's attention: non-temporal stores
          const unsigned r = (unsigned)(wrow0 + row), sq = r / seq;
          bf16_t* dst = cache + ((((long long)eg * p.rope.batch + sq) * (p.rope.k / 128) + kv) * p.rope.cap + (r - sq * seq)) * 128 + j0;
          st_stream(dst, lo);
          st_stream(dst + 64, hi);
        }
      }
    } else if constexpr (EPI == EPI_ROWPAR) {
      if (en0 + bn_out <= p.hs) slabs(std::integral_constant<int, 1>{});
      else if (en0 >= p.hs) slabs(std::integral_constant<int, 2>{});
      else slabs(std::integral_constant<int, 0>{});
    } else {
      slabs(std::integral_constant<int, 0>{});
    }
    pid += pid_step;
    if (!CFG::PERSIST || pid >= pid_end) break;
    behind_stores = true;
  }
}

template <class CFG, bool AT, bool BT, int EPI>
__global__ __launch_bounds__(CFG::THREADS, CFG::MIN_WAVES_PER_EU) void gemm_kernel(const GemmParams p) {
  __shared__ uint4 smem[CFG::SMEM_CHUNKS];
  gemm_tiles<CFG, AT, BT, EPI>(p, smem, blockIdx.x, gridDim.x);
}

// Two GEMMs that do not depend on each other in one launch: the data gradient (NN) and the weight gradient (TN) that wait for
// the same tensor, with the sums of the norm's parameter gradients in front of them (n_sums workgroups, see norm_sums), or the
// private and the shared columns of a row-parallel product with the reduce inside (both NT).  Workgroups of the second one
// (the one with the shorter tiles) start wherever the first leaves a slot idle, and there are one or two launches less, each
// with a start, an end and a last round of its own.  n_sums and n_first are multiples of 8, so that a workgroup's number
// within its GEMM names its XCD.  256 tokens of h = 768, T = 2, ffn 3072: 6 launches of 39.4 us become 3 of 30.1; 1111
// tokens of 2048, T = 4, SwiGLU, ffn 5632: 204 -> 188 us; see gemm_pair.
template <class CFG, class P1, class P2>
__global__ __launch_bounds__(CFG::THREADS, CFG::MIN_WAVES_PER_EU) void gemm_pair_kernel(const GemmParams p1, const GemmParams p2,
                                                                                      const NormSums sums, int n_sums, int n_first,
                                                                                      int second_first) {
  __shared__ uint4 smem[CFG::SMEM_CHUNKS];
  int b = blockIdx.x;
  if constexpr (P1::BT) {
    if (b < n_sums) {
      norm_sums(sums, b, reinterpret_cast<float4*>(smem));
      return;
    }
    b -= n_sums;
  }
  const bool first = b < n_first;
  const int nb = first ? n_first : (int)gridDim.x - n_sums - n_first;
  if (!first) b -= n_first;
  if (first == (second_first != 0)) gemm_tiles<CFG, P2::AT, P2::BT, P2::EPI>(p2, smem, b, nb);
  else gemm_tiles<CFG, P1::AT, P1::BT, P1::EPI>(p1, smem, b, nb);
}
template <bool AT_, bool BT_, int EPI_>
struct GemmKind {   // operand layouts and epilogue
  static constexpr bool AT = AT_, BT = BT_;
  static constexpr int EPI = EPI_;
};

// workgroups for `total` tiles, 0 if there are too many or the device cannot be asked
template <class CFG>
static long long tile_blocks(long long total) {
  if (total <= 0 || total > 0x7FFFFFFFLL) return 0;
  if (!CFG::PERSIST) return total;
  static int n_cu = 0;  // as many workgroups as the compute units hold at once
  if (n_cu == 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return 0;
    n_cu = v > 0 ? v : 256;
  }
  return total < (long long)n_cu * CFG::WGS_PER_CU ? total : (long long)n_cu * CFG::WGS_PER_CU;
}

template <class CFG, bool AT, bool BT, int EPI>
static hipError_t launch_one(const GemmParams& p, hipStream_t s) {
  constexpr int BN_OUT = (EPI == EPI_SWIGLU_FWD) ? CFG::BN / 2 : CFG::BN;
  if (p.bn_out < 0 || p.bn_out > BN_OUT || (p.bn_out & 7)) return hipErrorInvalidValue;
  const long long bn_out = (CFG::STREAM_B && p.bn_out > 0) ? p.bn_out : BN_OUT;  // as in the kernel
  const long long tiles_m = (p.M + CFG::BM - 1) / CFG::BM;
  const long long tiles_n = (p.N + bn_out - 1) / bn_out;
  const long long blocks = tile_blocks<CFG>(tiles_m * tiles_n * p.G);
  if (blocks <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL((gemm_kernel<CFG, AT, BT, EPI>), dim3((unsigned)blocks), dim3(CFG::THREADS), 0, s, p);
  return hipGetLastError();
}

template <class CFG, class P1, class P2>
static hipError_t launch_pair_one(const GemmPair& pair, const GemmParams& p1, const GemmParams& p2, const NormSums& sums,
                                  hipStream_t s) {
  auto tiles = [](const GemmParams& p) {
    return ((long long)p.M + CFG::BM - 1) / CFG::BM * ((p.N + CFG::BN - 1) / CFG::BN) * p.G;
  };
  const bool sf = pair.second_first;
  const long long t1 = tiles(sf ? p2 : p1), t2 = tiles(sf ? p1 : p2);
  const long long b1 = tile_blocks<CFG>(t1), b2 = pair.one_each ? t2 : tile_blocks<CFG>(t2);
  if (b1 <= 0 || b2 <= 0 || b1 + b2 > 0x7FFF0000LL) return hipErrorInvalidValue;
  auto eights = [](long long v) { return ((unsigned)v + 7u) & ~7u; };
  const unsigned n_sums = P1::BT ? eights(norm_sums_blocks(sums)) : 0u, n_first = eights(b1), n_second = eights(b2);
  hipLaunchKernelGGL((gemm_pair_kernel<CFG, P1, P2>), dim3(n_sums + n_first + n_second), dim3(CFG::THREADS), 0, s, p1, p2, sums,
                     (int)n_sums, (int)n_first, sf ? 1 : 0);
  return hipGetLastError();
}

}  // namespace caat
