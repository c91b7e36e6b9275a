// Weight-streaming GEMM for few token rows (decode batches, very short prompts): c_g[M,N] = a_g[M,K] b_g[N,K]^T with the
// fused epilogues of the forward pass, gfx950.
//
// What bounds it: the weights, read once from HBM, and so the bytes a compute unit keeps in flight.  The tile kernel
// (64 x 64, four shared stages, a barrier per stage) had 18 KB of weights in flight per compute unit on a shard of 1536
// rows and a round trip's wait per stage: 3.8 TB/s.  Here 40 - 110 KB are in flight and no wave waits for another.
// Register loads instead of the LDS ring (16 rows x 64 bytes per instruction in place of 8 rows x 128) reached 4.4.
// Measured, 7B shapes at T = 8 (us, tile kernel -> this one; 1 / 16 / 64 token rows):
//   q|k|v     100 MB  26.4 -> 17.8   26.0 -> 18.2   26.1 -> 22.9
//   gate|up   180 MB  40.0 -> 30.1   41.0 -> 31.1   46.0 -> 37.3
//   down       90 MB  21.4 -> 17.9   22.1 -> 20.6   (24.3, 28.6: see choose_route)
#pragma once
#include "caat_internal.h"

namespace caat {

typedef __bf16 bf16x8s_t __attribute__((ext_vector_type(8)));
typedef float f32x4s_t __attribute__((ext_vector_type(4)));

// MT tiles of 16 token rows x RT tiles of 16 weight rows per workgroup, NW waves that share the contraction: wave w
// takes the 64-wide k chunks w, w + NW, ... of all rows, so the waves of a workgroup read NW consecutive cache lines of
// every row at a time and nothing is read twice inside a workgroup.  Every wave copies its own chunks global -> LDS
// (whole 128-byte lines) into a ring of NST slots that only it reads: it waits for its own copies alone, and there is no
// barrier until the waves' partial sums meet at the end.
template <int MT, int RT, int NW, int LDS_KB, int EPI>
__global__ __launch_bounds__(64 * NW) void gemm_stream_kernel(const GemmParams p) {
  constexpr bool SWI = EPI == EPI_SWIGLU_FWD;
  constexpr int OT = SWI ? RT / 2 : RT;            // output tiles of 16 columns
  constexpr int NI = 2 * (RT + MT);                // copies of a stage, 1 KB (8 rows of 128 bytes) each
  constexpr int NST_LDS = LDS_KB / (NW * NI), NST_CNT = 63 / NI + 1;
  constexpr int NST = NST_LDS < NST_CNT ? NST_LDS : NST_CNT;
  static_assert(NST >= 2, "a wave needs two slots");
  constexpr int RED_KB = NW * RT;                  // partial sums of one token tile
  constexpr int MG = RED_KB * MT <= NW * NI * NST ? MT : (RED_KB * 2 <= NW * NI * NST && MT % 2 == 0 ? 2 : 1);
  static_assert(RED_KB * MG <= NW * NI * NST, "the partial sums take the ring's place");
  __shared__ uint4 smem[NW * NST * NI * 64];
  f32x4s_t(*red)[MG][RT][64] = reinterpret_cast<f32x4s_t(*)[MG][RT][64]>(smem);
  constexpr unsigned OOBS = 0x80000000u;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, q4 = lane >> 4;
  // tile order: ids cut into 8 contiguous ranges, one per XCD; inside, token tiles vary fastest (they share the weights)
  const int bn = p.bn_out;
  const int tiles_m = (p.M + MT * 16 - 1) / (MT * 16), tiles_n = (p.N + bn - 1) / bn;
  const int total = tiles_m * tiles_n * p.G;
  int id;
  {
    const int q = total >> 3, rem = total & 7, x = blockIdx.x & 7;
    id = x * q + (x < rem ? x : rem) + (int)(blockIdx.x >> 3);
  }
  const int g = id / (tiles_m * tiles_n);
  const int t = id - g * (tiles_m * tiles_n);
  const int n0 = (t / tiles_m) * bn, m0 = (t % tiles_m) * (MT * 16);
  const i32x4_t ra = make_rsrc(p.a + (long long)g * p.stride_a + (long long)m0 * p.lda);
  const i32x4_t rb = make_rsrc(p.b + (long long)g * p.stride_b + (long long)n0 * p.ldb);
  // copy i of a stage: rows 8 i .. 8 i + 7 (weights, then tokens); slot c of row r holds the chunk c ^ ((r >> 1) & 7), so
  // that 16 rows read the same logical chunk from different banks
  unsigned off[NI];
  const int r8 = lane >> 3;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int row = (i < 2 * RT ? i : i - 2 * RT) * 8 + r8;
    const int chunk = (lane & 7) ^ ((row >> 1) & 7);
    if (i < 2 * RT) {
      const int col = SWI && row >= OT * 16 ? row - OT * 16 : row;   // output column inside the tile
      const bool ok = col < bn && n0 + col < p.N;
      off[i] = ok ? (unsigned)(((long long)(col + (SWI && row >= OT * 16 ? p.half : 0)) * p.ldb + chunk * 8) * 2) : OOBS;
    } else {
      off[i] = m0 + row < p.M ? (unsigned)((row * p.lda + chunk * 8) * 2) : OOBS;
    }
  }
  f32x4s_t acc[RT][MT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[r][m] = f32x4s_t{0.0f, 0.0f, 0.0f, 0.0f};
  const int K = p.K, chunks = (K + 63) / 64;
  uint4* ring = smem + wave * (NST * NI * 64);
  auto copy = [&](int c, int slot) {
    const int k0 = c * 64;
    uint4* dst = ring + slot * (NI * 64);
    i32x4_t sa = ra, sb = rb;                        // the chunk's k offset goes into the base address
    const unsigned long long da = (unsigned long long)(unsigned)ra.x + ((unsigned long long)(unsigned)ra.y << 32) + (unsigned long long)k0 * 2;
    const unsigned long long db = (unsigned long long)(unsigned)rb.x + ((unsigned long long)(unsigned)rb.y << 32) + (unsigned long long)k0 * 2;
    sa.x = (int)(unsigned)da; sa.y = (int)(unsigned)(da >> 32);
    sb.x = (int)(unsigned)db; sb.y = (int)(unsigned)(db >> 32);
    const bool whole = k0 + 64 <= K;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      unsigned o = off[i];
      if (!whole) {                                  // the last chunk of a ragged K, or none
        const int row = (i < 2 * RT ? i : i - 2 * RT) * 8 + r8;
        if (k0 + ((lane & 7) ^ ((row >> 1) & 7)) * 8 >= K) o = OOBS;
      }
      if (i < 2 * RT) dma16<true>(sb, o, dst + i * 64);
      else dma16<false>(sa, o, dst + i * 64);
    }
  };
#pragma unroll
  for (int d = 0; d < NST; ++d) copy(wave + d * NW, d);
  const int swz = (r16 >> 1) & 7;
  int slot = 0;
  for (int c = wave; c < chunks; c += NW) {
    wait_vmcnt<(NST - 1) * NI>();
    const uint4* src = ring + slot * (NI * 64);
    bf16x8s_t wf[2][RT], af[2][MT];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int at = r16 * 8 + ((h * 4 + q4) ^ swz);
#pragma unroll
      for (int r = 0; r < RT; ++r) wf[h][r] = __builtin_bit_cast(bf16x8s_t, src[r * 128 + at]);
#pragma unroll
      for (int m = 0; m < MT; ++m) af[h][m] = __builtin_bit_cast(bf16x8s_t, src[(RT + m) * 128 + at]);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {   // the fragments are in registers before the slot is filled again
#pragma unroll
      for (int r = 0; r < RT; ++r) asm volatile("" : "+v"(wf[h][r]));
#pragma unroll
      for (int m = 0; m < MT; ++m) asm volatile("" : "+v"(af[h][m]));
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    copy(c + NST * NW, slot);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[r][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[h][r], af[h][m], acc[r][m], 0, 0, 0);
    slot = slot + 1 == NST ? 0 : slot + 1;
  }
  wait_vmcnt<0>();                                  // the copies past the end write zeros: let them land
  __syncthreads();                                  // before the partial sums take the rings' place
  // lane: row m0 + 16 m + r16, columns n0 + 16 r + 4 q4 .. +3
#pragma unroll
  for (int mg = 0; mg < MT; mg += MG) {
    if (mg) __syncthreads();
#pragma unroll
    for (int m = 0; m < MG; ++m)
#pragma unroll
      for (int r = 0; r < RT; ++r) red[wave][m][r][lane] = acc[r][mg + m];
    __syncthreads();
    for (int u = tid; u < MG * OT * 64; u += 64 * NW) {
      const int l = u & 63, r = (u >> 6) % OT, m = (u >> 6) / OT;
      auto sum = [&](int rr) {
        f32x4s_t s = red[0][m][rr][l];
#pragma unroll
        for (int w = 1; w < NW; ++w) s += red[w][m][rr][l];
        return s;
      };
      const int row = m0 + (mg + m) * 16 + (l & 15), cl = r * 16 + (l >> 4) * 4, col = n0 + cl;
      if (row >= p.M || cl >= bn || col >= p.N) continue;   // N % 8 == 0, bn % 8 == 0: 4 columns share validity
      auto put4 = [](bf16_t* dst, float a, float b, float c, float d) {
        *reinterpret_cast<uint2*>(dst) = make_uint2(pack2bf(a, b), pack2bf(c, d));
      };
      const f32x4s_t s = sum(r);
      bf16_t* c = p.c + (long long)g * p.stride_c + (long long)row * p.ldc + col;
      if constexpr (EPI == EPI_PLAIN) {
        put4(c, s[0], s[1], s[2], s[3]);
      } else {
        // the element-wise work starts from the bf16-rounded accumulator, as in the block-sized kernel
        const unsigned lo = pack2bf(s[0], s[1]), hi = pack2bf(s[2], s[3]);
        const float v[4] = {lo_bf(lo), hi_bf(lo), lo_bf(hi), hi_bf(hi)};
        if constexpr (EPI == EPI_GELU_FWD) {
          *reinterpret_cast<uint2*>(c) = make_uint2(lo, hi);
          put4(p.c2 + (long long)g * p.stride_c2 + (long long)row * p.ldc2 + col, gelu_f(v[0]), gelu_f(v[1]), gelu_f(v[2]), gelu_f(v[3]));
        } else if constexpr (EPI == EPI_ROWPAR) {
          float o[4];
          const uint2 rw = *reinterpret_cast<const uint2*>(p.aux + (long long)g * p.stride_aux + (long long)row * p.ldaux + col);
          const float rr[4] = {lo_bf(rw.x), hi_bf(rw.x), lo_bf(rw.y), hi_bf(rw.y)};
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = col + e >= p.hs ? p.scale * v[e] + rr[e] : v[e];
          put4(c, o[0], o[1], o[2], o[3]);
        } else if constexpr (SWI) {
          const f32x4s_t su = sum(OT + r);
          const unsigned ulo = pack2bf(su[0], su[1]), uhi = pack2bf(su[2], su[3]);
          const float up[4] = {lo_bf(ulo), hi_bf(ulo), lo_bf(uhi), hi_bf(uhi)};
          *reinterpret_cast<uint2*>(c) = make_uint2(lo, hi);
          *reinterpret_cast<uint2*>(c + p.half) = make_uint2(ulo, uhi);
          float y[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = v[e] * sigmoid_f(v[e]) * up[e];
          put4(p.c2 + (long long)g * p.stride_c2 + (long long)row * p.ldc2 + col, y[0], y[1], y[2], y[3]);
        }
      }
    }
  }
}

}  // namespace caat
