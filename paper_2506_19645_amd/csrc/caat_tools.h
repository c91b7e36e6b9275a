/*
 * caat_tools.h -- measuring tools that libcaat.so exports next to the method's C ABI (include/caat.h).  They are not
 * part of the method: bench.py binds them to time every launch of a block call and to probe HBM streaming rates.
 */
#ifndef CAAT_TOOLS_H
#define CAAT_TOOLS_H

#include <stddef.h>

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Per-launch timing of the block calls (a host-side measuring tool, not part of the method): while enabled,
 * caat_block_fwd / caat_block_bwd bracket every kernel they enqueue with a pair of HIP events on the caller's
 * stream.  caat_profile_get waits for record `index` (in launch order since the last reset) and returns a
 * static kernel-family name (host pointer to a NUL-terminated string) and the elapsed milliseconds.  Events
 * are created on first use and reused after a reset.  Not thread-safe; off by default.
 * on = 2: the kernels of an untimed call, so the same results; two GEMMs in one launch (caat_gemm_pair_route,
 * caat_gemm_shared_pair_route) are one record named after both, "a+b".
 * on = 1: every GEMM a launch of its own, so that each has a time, and the rotation of q and k a pass of its own.  Other kernels
 * run then, and low-order bits may differ from an untimed call's: a gradient's contraction may be split between two groups of
 * waves, and the rotation takes every angle's sine and cosine itself (in the product's epilogue most are turned on from 16 rows
 * before), so the gradients, the projections, the caches and what follows from them.
 */
int caat_profile_enable(int on);
int caat_profile_reset(void);
int caat_profile_count(void);
int caat_profile_get(int index, const char** name, float* ms);

/*
 * HBM streaming probe (a measuring tool, not part of the method): enqueues one kernel that reads `bytes` bytes of
 * the device buffer `src` (16-byte aligned, bytes % 16 == 0) and, for the copy modes, writes them to `dst`.
 *   mode 0: read, every workgroup walks its own contiguous piece, plain loads
 *   mode 1: the same with the non-temporal hint on the loads
 *   mode 2: read, the whole grid sweeps one window (grid-stride), plain loads
 *   mode 3: copy src -> dst, contiguous piece per workgroup, plain loads and stores
 *   mode 4: the same with the non-temporal hint on loads and stores
 * dst may be NULL for the read modes (a result is only stored if the data hash to one particular value, which
 * keeps the loads alive; pass a buffer of at least 16 bytes to be safe).  The caller times it with events on
 * `hip_stream`; bench.py --probe-hbm does.  This is where the cache-policy choices of the streaming kernels
 * (which accesses carry the hint) were measured.
 */
int caat_hbm_probe(const void* src, void* dst, size_t bytes, int mode, void* hip_stream);

/*
 * Which kernel a shard GEMM of these sizes runs on (host only, nothing is launched), for tests that mean to reach every
 * kernel and for traces.  layout: caat_gemm_layout; epilogue: 0 plain, 1 GELU, 2 SwiGLU, 3 row-parallel, 4 GELU', 5
 * SwiGLU', 6 the shared channels of `ranks` ranks (G = 1); shard_cols: for 3, the columns of the whole shard where N is a
 * part of them (0 = N).  Returns
 *   0 .. 7   tile of 256 x 256, 192 x 256, 256 x 192, 128 x 128, 64 x 128, 64 x 64, and 128 x 128, 64 x 64 by two wave groups
 *   8        the tile for few token rows that meet many weight rows
 *   16 mt + rt (+ 128)   the weight-streaming kernel, 16 mt token rows x 16 rt weight rows per workgroup (128: of two waves)
 *   256 g + tile         6 only: fp32 sums over g groups of ranks on that tile, then a kernel that adds them up
 * or -1 for arguments out of range.
 */
int caat_gemm_route(int layout, int epilogue, int G, long long M, long long N, long long K, int ranks, long long shard_cols);

/*
 * How the backward enqueues a data gradient [M, N] of contraction K and the weight gradient [K, N] of contraction M that goes
 * with it, for G ranks (host only): -1 one after the other (caat_gemm_route names the kernels), else in one launch: tile 0, 1,
 * 3, 4 or 5 of caat_gemm_route, + 16 where the weight gradient's tiles come first, + 32 where a workgroup of the second of
 * them takes one tile and not a share of several.  -2 for arguments out of range.
 */
int caat_gemm_pair_route(int G, long long M, long long N, long long K);

/*
 * The same for the row-parallel product of reduce_in_gemm, M tokens of contraction K per rank (host only): -1 the private and
 * the shared columns one after the other, else caat_gemm_pair_route's numbers (the shared columns in place of the weight
 * gradient) + 256 times the groups of ranks that the shared columns are summed in, with all the scratch that helps.
 */
int caat_gemm_shared_pair_route(int T, long long M, long long h, long long hs, long long K);

#ifdef __cplusplus
}
#endif
#endif /* CAAT_TOOLS_H */
