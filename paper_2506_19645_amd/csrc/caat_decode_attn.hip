// Decode attention for gfx950: one new token per sequence at position kv_len, the attention of its query heads over the
// kv_len cached keys and its own; RoPE of q and the new k and the append to the caches in the same launch.
//
// What bounds it: the K / V rows, read once from HBM.  A workgroup owns one (rank, sequence, key / value head) with ALL
// query heads of its group (up to 16; more are covered by further workgroups) and one of `splits` ranges of keys, so
// grouped-query heads share one pass over the rows and a small batch still fills the chip.  Its waves take 16-key blocks
// in turn; every wave copies its blocks global -> LDS (whole rows) into two slots that only it reads, waits for its own
// copies alone, and computes S = K q^T and O^T += V^T P with MFMAs (columns = query heads; most are idle for multi-head
// attention, but the matrix unit has nothing else to do).  P goes in as an exact sum of three bf16 values, so the result is
// that of fp32 probabilities; a wave whose sums are not finite (infinity less infinity inside such a sum) repeats its keys
// with fp32 MFMAs, which as the only path cost a decode layer 2 to 4 %.  The waves' partial results meet in
// LDS in a fixed order, the ranges' in a second small kernel.
// Against one workgroup per query head that streamed its rows through registers (us, before -> now): batch 64, 32 heads,
// 2048 keys 317 -> 312 (6.9 TB/s); batch 1, 3001 keys 51.5 -> 18; batch 16, 64 query / 8 key heads, 1999 keys 160 -> 31;
// batch 32, 32 / 8 heads, 4000 keys 314 -> 85; batch 100, 16 heads, 300 keys 47 -> 47.  Two waves, or blocks of 32 keys,
// or three and four slots per wave were up to 8 % slower at batch 64 or up to 40 % on short caches.
#include <math.h>
#include <algorithm>
#include <type_traits>
#include "caat_internal.h"

namespace caat {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4_t* lds_s4_t;
typedef __attribute__((address_space(3))) const char* lds_c_t;

static constexpr int DHD = 128;                  // head dim
static constexpr int DKB = 16;                   // keys per block
static constexpr int DNW = 4;                    // waves per workgroup, DNS slots each: 64 KB, two workgroups per compute unit
static constexpr int DNS = 2;
static constexpr int DNI = 8;                    // 1 KB copies per block: 4 of K, 4 of V (4 rows of 256 bytes each)

// LDS slot: K block [16 rows][16 chunks of 16 bytes], then the V block.  K is read 16 rows x one chunk at a time, V by
// the transpose read, 8 rows x two chunks for 32 lanes: each spread over all banks by its own swizzle.
__device__ __forceinline__ int dk_swz(int row) { return row & 15; }
__device__ __forceinline__ int dv_swz(int row) { return (row & 7) << 1; }

// qkv holds the UN-rotated projections of the token at position nkeys - 1; q and the new k are rotated here (rounded to
// bf16 as the RoPE kernels store them), the new k and v take part from registers and are written to cache row nkeys - 1,
// which nobody reads in this launch.
__global__ __launch_bounds__(64 * DNW) void decode_attn_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ kc,
                                                               bf16_t* __restrict__ vc, bf16_t* __restrict__ out,
                                                               float* __restrict__ part, int hpr, int kvpr, long long cap,
                                                               int nkeys, float scale_log2, float log2_base, int splits) {
  __shared__ uint4 ring[DNW * DNS * DNI * 64];
  static_assert(DNW * 16 * (DHD + 4) * 4 <= DNW * DNS * DNI * 1024, "the partial results take the rings' place");
  __shared__ uint4 s_q[18 * 16];                 // query heads, then the new key and value, 16 chunks each
  __shared__ float s_cs[64], s_sn[64];
  __shared__ float s_m[DNW][16], s_l[DNW][16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int grp = hpr / kvpr, qtiles = (grp + 15) / 16;
  int u = blockIdx.x;
  const int split = u % splits;
  u /= splits;
  const int qt = u % qtiles;
  u /= qtiles;                                   // sequence * kvpr + key / value head
  const long long sq = u / kvpr;
  const int kvh = (int)(u - sq * kvpr);
  const int nq = min(16, grp - qt * 16);         // query heads of this workgroup
  const int head0 = kvh * grp + qt * 16;         // the first, inside the rank
  const bf16_t* kbase = kc + (long long)u * cap * DHD;
  const bf16_t* vbase = vc + (long long)u * cap * DHD;
  const int ncache = nkeys - 1;                  // keys that come from the caches
  const int nb = (nkeys + DKB - 1) / DKB;        // blocks; the new key sits in the last one
  const int b0 = (int)((long long)nb * split / splits), b1 = (int)((long long)nb * (split + 1) / splits);

  uint4* mine = ring + wave * (DNS * DNI * 64);
  auto copy = [&](int b, int slot) {
    const int key0 = b * DKB;
    const bool any = b < b1;
    const i32x4_t rk = make_rsrc(kbase + (long long)(any ? key0 : 0) * DHD), rv = make_rsrc(vbase + (long long)(any ? key0 : 0) * DHD);
    uint4* dst = mine + slot * (DNI * 64);
    const int left = any ? ncache - key0 : 0;    // cached keys from this block on
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = i * 4 + g;
      const bool ok = row < left;
      dma16<true>(rk, ok ? (unsigned)(row * 256 + ((r16 ^ dk_swz(row)) << 4)) : 0x80000000u, dst + i * 64);
      dma16<true>(rv, ok ? (unsigned)(row * 256 + ((r16 ^ dv_swz(row)) << 4)) : 0x80000000u, dst + (4 + i) * 64);
    }
  };
  // Projections of the token: four query heads per wave (one copy), new key and value (wave 0) ...
  const bf16_t* row = qkv + sq * (long long)(hpr + 2 * kvpr) * DHD;
  {
    const int hd = wave * 4 + g;
    static_assert(DNW == 4, "four query heads per wave");
    dma16(make_rsrc(row + (long long)head0 * DHD), hd < nq ? (unsigned)(hd * 256 + r16 * 16) : 0x80000000u, s_q + wave * 64);
    if (wave == 0 && lane < 32)
      dma16(make_rsrc(row + (long long)(hpr + kvh) * DHD), (unsigned)(g * kvpr * 256 + r16 * 16), s_q + 16 * 16);
  }
  // ... then the first keys are on their way while q is prepared
#pragma unroll
  for (int i = 0; i < DNS; ++i) copy(b0 + wave + i * DNW, i);
  if (tid < 64) {
    // angle j of the position, j = 0 .. 63, once per workgroup (the RoPE kernels' sine and cosine)
    float sn, cs;
    rope_sincos((float)(nkeys - 1), rope_freq(tid, 128, log2_base), sn, cs);
    s_cs[tid] = cs;
    s_sn[tid] = sn;
  }
  wait_vmcnt<DNS * DNI>();                       // the projections have landed
  __syncthreads();
  bf16x8_t qf[4];                                // lane: query head r16, dims 32 ks + 8 g .. + 7
  uint4 knew = make_uint4(0u, 0u, 0u, 0u), vnew = knew;   // the token's own key (rotated) and value: dims 8 r16 .. + 7
  {
    uint4 qw[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) qw[ks] = s_q[r16 * 16 + ks * 4 + g];   // heads past nq were filled with zeros
    const uint4 kw = s_q[16 * 16 + r16];
    vnew = s_q[17 * 16 + r16];
    // q: the pairs (j, j + 64) of a lane's 8 dims are its slices ks and ks + 2
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const unsigned x1[4] = {qw[ks].x, qw[ks].y, qw[ks].z, qw[ks].w}, x2[4] = {qw[ks + 2].x, qw[ks + 2].y, qw[ks + 2].z, qw[ks + 2].w};
      unsigned y1[4], y2[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float a[2], b[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float cs = s_cs[ks * 32 + g * 8 + i * 2 + e], sn = s_sn[ks * 32 + g * 8 + i * 2 + e];
          const float p = e ? hi_bf(x1[i]) : lo_bf(x1[i]), q = e ? hi_bf(x2[i]) : lo_bf(x2[i]);
          a[e] = p * cs - q * sn;
          b[e] = q * cs + p * sn;
        }
        y1[i] = pack2bf(a[0], a[1]);
        y2[i] = pack2bf(b[0], b[1]);
      }
      qw[ks] = make_uint4(y1[0], y1[1], y1[2], y1[3]);
      qw[ks + 2] = make_uint4(y2[0], y2[1], y2[2], y2[3]);
    }
    // the new key: lane r16 holds dims 8 r16 .. + 7, its pair is 8 lanes away
    {
      const unsigned own[4] = {kw.x, kw.y, kw.z, kw.w};
      unsigned res[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned oth = (unsigned)__shfl_xor((int)own[i], 8, 64);
        float y[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int j = (r16 & 7) * 8 + i * 2 + e;
          const float a = e ? hi_bf(own[i]) : lo_bf(own[i]), b = e ? hi_bf(oth) : lo_bf(oth);
          const float cs = s_cs[j], sn = s_sn[j];
          y[e] = r16 < 8 ? a * cs - b * sn : a * cs + b * sn;
        }
        res[i] = pack2bf(y[0], y[1]);
      }
      knew = make_uint4(res[0], res[1], res[2], res[3]);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) qf[ks] = __builtin_bit_cast(bf16x8_t, qw[ks]);
  }

  f32x4_t acc[8];                                // O^T: dims 16 dt + 4 g + 0..3, query head r16
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) acc[dt] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  float m = -INFINITY, l = 0.0f;                 // l: this lane's keys only
  auto sweep = [&](auto fp32_c) {                // the wave's blocks; the first DNS copies are under way
    int slot = 0;
    for (int b = b0 + wave; b < b1; b += DNW) {
      wait_vmcnt<(DNS - 1) * DNI>();             // this block has landed; the next ones may be in flight
      uint4* ks = mine + slot * (DNI * 64);
      uint4* vs = ks + 4 * 64;
      if (b == nb - 1 && g == 0) {               // the token's own key and value take their row of the last block
        const int r = (nkeys - 1) & (DKB - 1);
        ks[r * 16 + (r16 ^ dk_swz(r))] = knew;
        vs[r * 16 + (r16 ^ dv_swz(r))] = vnew;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      bf16x8_t kf[4];
      short4_t vf[8];
#pragma unroll
      for (int t = 0; t < 4; ++t) kf[t] = __builtin_bit_cast(bf16x8_t, ks[r16 * 16 + ((t * 4 + g) ^ dk_swz(r16))]);
      const int vr = 4 * g + (r16 >> 2);         // the keys of this lane's scores are 4 g .. 4 g + 3
      const lds_c_t va = (lds_c_t)vs + vr * 256 + (r16 & 1) * 8;
#pragma unroll
      for (int dt = 0; dt < 8; ++dt)
        vf[dt] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_t)(va + (((dt * 2 + ((r16 & 3) >> 1)) ^ dv_swz(vr)) << 4)));
#pragma unroll
      for (int t = 0; t < 4; ++t) asm volatile("" : "+v"(kf[t]));
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) asm volatile("" : "+v"(vf[dt]));
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the fragments are in registers before the slot is filled again
      copy(b + DNS * DNW, slot);
      f32x4_t sc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int t = 0; t < 4; ++t) sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[t], qf[t], sc, 0, 0, 0);
      // scores of query head r16 and keys 16 b + 4 g + r
      float p[4], mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p[i] = sc[i] * scale_log2;
        if (b * DKB + 4 * g + i >= nkeys) p[i] = -INFINITY;
        mx = fmaxf(mx, p[i]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m, mx);          // every block holds a key below nkeys: -inf only if all its scores are
      const float alpha = exp2f(m - m_new);      // 0 in the first block
      float sum = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p[i] = exp2f(p[i] - m_new);
        sum += p[i];
      }
      l = l * alpha + sum;
      m = m_new;
#pragma unroll
      for (int dt = 0; dt < 8; ++dt)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[dt][r] *= alpha;
      if constexpr (decltype(fp32_c)::value) {
#pragma unroll
        for (int i = 0; i < 4; ++i)              // step i of the product: the keys 4 g + i, g = 0 .. 3
#pragma unroll
          for (int dt = 0; dt < 8; ++dt)
            acc[dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf2f((bf16_t)vf[dt][i]), p[i], acc[dt], 0, 0, 0);
      } else {
        unsigned hi[2], mid[2], lo[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          hi[i] = pack2bf(p[2 * i], p[2 * i + 1]);
          const float a = p[2 * i] - lo_bf(hi[i]), c = p[2 * i + 1] - hi_bf(hi[i]);   // exact, as is the next difference
          mid[i] = pack2bf(a, c);
          lo[i] = pack2bf(a - lo_bf(mid[i]), c - hi_bf(mid[i]));
        }
        const bf16x8_t ph = __builtin_bit_cast(bf16x8_t, make_uint4(hi[0], hi[1], mid[0], mid[1]));
        const short4_t pl = __builtin_bit_cast(short4_t, make_uint2(lo[0], lo[1]));
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {           // one product takes the first two parts against the values twice
          const uint2 v = __builtin_bit_cast(uint2, vf[dt]);
          const bf16x8_t v2 = __builtin_bit_cast(bf16x8_t, make_uint4(v.x, v.y, v.x, v.y));
          acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v2, ph, acc[dt], 0, 0, 0);
        }
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) acc[dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf[dt], pl, acc[dt], 0, 0, 0);
      }
      slot = slot + 1 == DNS ? 0 : slot + 1;
    }
  };
  sweep(std::false_type{});
  wait_vmcnt<0>();                               // the copies past the end write zeros: let them land
  bool odd = false;
#pragma unroll
  for (int dt = 0; dt < 8; ++dt)
#pragma unroll
    for (int r = 0; r < 4; ++r) odd |= !(fabsf(acc[dt][r]) < INFINITY);
  if (__any(odd)) {
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) acc[dt] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    m = -INFINITY;
    l = 0.0f;
#pragma unroll
    for (int i = 0; i < DNS; ++i) copy(b0 + wave + i * DNW, i);
    sweep(std::true_type{});
    wait_vmcnt<0>();
  }
  if (qt == 0 && split == splits - 1 && wave == 0 && g == 0) {   // one 16-lane group writes the new rows of the caches
    const long long dst = ((long long)u * cap + (nkeys - 1)) * DHD + r16 * 8;
    st_stream(kc + dst, knew);
    st_stream(vc + dst, vnew);
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  __syncthreads();                               // before the partial results take the rings' place
  constexpr int HS = DHD + 4;                    // floats per head row (padded)
  float* po = reinterpret_cast<float*>(ring);    // [DNW][16][HS]
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) *reinterpret_cast<f32x4_t*>(po + (wave * 16 + r16) * HS + dt * 16 + 4 * g) = acc[dt];
  if (g == 0) {
    s_m[wave][r16] = m;
    s_l[wave][r16] = l;
  }
  __syncthreads();
  for (int i = tid; i < nq * DHD; i += 64 * DNW) {
    const int hd = i / DHD, d = i - hd * DHD;
    float M = s_m[0][hd];
#pragma unroll
    for (int w = 1; w < DNW; ++w) M = fmaxf(M, s_m[w][hd]);
    float num = 0.0f, den = 0.0f;
#pragma unroll
    for (int w = 0; w < DNW; ++w) {
      const float f = exp2f(s_m[w][hd] - M);     // 0 for a wave without a block
      num += po[(w * 16 + hd) * HS + d] * f;
      den += s_l[w][hd] * f;
    }
    const long long h = sq * hpr + head0 + hd;
    if (splits == 1) {
      out[h * DHD + d] = f2bf(num / den);
    } else {                                     // [query head][split][128 sums | maximum | denominator | 2 unused]
      float* dst = part + (h * splits + split) * HS;
      dst[d] = num;
      if (d == 0) {
        dst[DHD] = M;
        dst[DHD + 1] = den;
      }
    }
  }
}

// the ranges of keys of one query head: their weights, then the sums in ascending order
static constexpr int DMAX_SPLITS = 64;
static constexpr long long DMAX_WGS = 1024;      // workgroups of a launch with more than one range: two rounds
__global__ __launch_bounds__(128) void decode_merge_kernel(const float* __restrict__ part, bf16_t* __restrict__ out, int splits) {
  __shared__ float s_f[DMAX_SPLITS];
  const int d = threadIdx.x, lane = d & 63;
  const float* p = part + (long long)blockIdx.x * splits * (DHD + 4);
  const bool have = lane < splits;               // every wave weighs the (at most 64) ranges
  const float m = have ? p[lane * (DHD + 4) + DHD] : -INFINITY, l = have ? p[lane * (DHD + 4) + DHD + 1] : 0.0f;
  float M = m;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, 64));
  const float f = exp2f(m - M);
  float den = l * f;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) den += __shfl_xor(den, off, 64);
  if (d < 64) s_f[d] = f;                        // 0 beyond the last range
  __syncthreads();
  float num = 0.0f;
  for (int s0 = 0; s0 < splits; s0 += 8) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = s0 + i < splits ? p[(s0 + i) * (DHD + 4) + d] : 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) num += v[i] * s_f[s0 + i];
  }
  out[(long long)blockIdx.x * DHD + d] = f2bf(num / den);
}

// Number of key ranges per (sequence, key / value head).  512 workgroups run at a time (two per compute unit) and together
// take about 830 blocks per microsecond (6.8 TB/s), one by itself at most about 3 (four waves, two blocks each per trip
// to memory); starting and finishing costs a workgroup about 3 us and the second kernel a launch about 4.5.
// `most`: as many as the scratch holds.
static int decode_splits(long long units, long long nkeys, long long most) {
  const long long nb = (nkeys + DKB - 1) / DKB;
  int best = 1;
  double cost = 0.0;
  for (int s = 1; s <= DMAX_SPLITS && (s == 1 || (s <= most && nb / s >= DNW && units * s <= DMAX_WGS)); ++s) {
    const long long wgs = units * s;
    const double rate = wgs < 277 ? 3.0 : 830.0 / (double)(wgs < 512 ? wgs : 512);   // blocks per us and workgroup
    const double c = (double)((wgs + 511) / 512) * ((double)((nb + s - 1) / s) / rate + 3.0) + (s > 1 ? 4.5 : 0.0);
    if (s == 1 || c < cost) {
      cost = c;
      best = s;
    }
  }
  return best;
}

// What any number of keys can take: it neither depends on it, so that one scratch serves a sequence as it grows, nor falls
// with the number of sequences.
size_t decode_attn_scratch_bytes(long long n_seq, int hpr, int kvpr) {
  const long long grp = hpr / kvpr, qtiles = (grp + 15) / 16, heads = (grp + qtiles - 1) / qtiles;
  const long long rows = std::min(n_seq * hpr * DMAX_SPLITS, DMAX_WGS * heads);   // heads: of one workgroup, at most
  return (size_t)rows * (DHD + 4) * sizeof(float);
}

// out [n_seq, hpr*128] = softmax(q K^T / sqrt(d)) V over keys 0 .. nkeys-1 of caches [n_seq][kvpr][cap][128].
// qkv as above; rope_base > 0.
hipError_t launch_decode_attn(const bf16_t* qkv, bf16_t* kc, bf16_t* vc, bf16_t* out, long long n_seq, int hpr,
                              int kvpr, int d, long long cap, long long nkeys, float rope_base, void* scratch, size_t scratch_bytes,
                              hipStream_t s) {
  if (d != DHD || kvpr < 1 || hpr % kvpr != 0 || nkeys < 1 || nkeys > cap || cap * 256 >= 0x7FFFFFFFLL || !(rope_base > 0.0f))
    return hipErrorInvalidValue;
  if (n_seq * hpr == 0) return hipSuccess;
  const long long units = n_seq * kvpr * ((hpr / kvpr + 15) / 16);
  const long long row = (DHD + 4) * (long long)sizeof(float);
  const int splits = decode_splits(units, nkeys, scratch ? (long long)scratch_bytes / (n_seq * hpr * row) : 1);
  if (units * splits > 0x7FFFFFFFLL || n_seq * hpr > 0x7FFFFFFFLL) return hipErrorInvalidValue;
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)d);
  const dim3 grid((unsigned)(units * splits)), wg(64 * DNW);
  float* part = reinterpret_cast<float*>(scratch);
  hipLaunchKernelGGL(decode_attn_kernel, grid, wg, 0, s, qkv, kc, vc, out, part, hpr, kvpr, cap, (int)nkeys, scale_log2,
                     log2f(rope_base), splits);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || splits == 1) return e;
  hipLaunchKernelGGL(decode_merge_kernel, dim3((unsigned)(n_seq * hpr)), dim3(128), 0, s, part, out, splits);
  return hipGetLastError();
}

}  // namespace caat
