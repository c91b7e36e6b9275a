"""Which kernel a shard GEMM runs on, asked on the host: the rules at the sizes where both sides were timed."""
import pytest

from paper_2506_19645_amd import binding as B

PLAIN, GELU, SWIGLU, ROWPAR = 0, 1, 2, 3


@pytest.mark.parametrize("epilogue,G,N,K,M,streams", [
    (PLAIN, 8, 1536, 4096, 96, True), (ROWPAR, 8, 1536, 2048, 128, True), (PLAIN, 8, 768, 4096, 65, True),   # one round
    (SWIGLU, 8, 1376, 4096, 96, True),                                    # two rounds of the widest, a long contraction
    (ROWPAR, 8, 1024, 5504, 65, False), (ROWPAR, 8, 2048, 1376, 96, False), (GELU, 8, 1728, 5120, 96, False),
    (SWIGLU, 4, 3584, 4096, 96, False), (ROWPAR, 8, 3072, 2048, 128, False), (SWIGLU, 8, 1728, 5120, 128, False),
    (SWIGLU, 8, 1376, 4096, 64, True), (ROWPAR, 8, 3072, 2048, 64, False), (SWIGLU, 8, 1728, 5120, 64, False),
    (SWIGLU, 4, 3584, 4096, 32, True), (SWIGLU, 4, 3584, 4096, 48, False), (SWIGLU, 8, 1376, 4096, 48, True),
    (SWIGLU, 8, 1728, 5120, 32, False), (SWIGLU, 8, 1728, 5120, 48, False), (ROWPAR, 8, 4096, 1376, 48, False), (ROWPAR, 8, 4096, 1376, 16, True),
    (PLAIN, 8, 1920, 5120, 48, False), (GELU, 8, 1728, 5120, 33, False), (ROWPAR, 8, 2048, 1376, 48, False),   # 64 x 64 tiles
    (GELU, 8, 1728, 5120, 32, True), (GELU, 8, 1728, 5120, 49, True), (PLAIN, 8, 1536, 4096, 48, True), (SWIGLU, 4, 2048, 3072, 48, True),
    (SWIGLU, 8, 1728, 5120, 1, False), (SWIGLU, 8, 1728, 5120, 16, False), (SWIGLU, 4, 3584, 512, 8, False), (GELU, 8, 3456, 5120, 1, True),
    (SWIGLU, 8, 1792, 4096, 1, True), (SWIGLU, 8, 1376, 4104, 1, True),
    (PLAIN, 1, 8, 8, 129, False)])
def test_few_token_rows_stream_the_weights_where_that_is_faster(epilogue, G, N, K, M, streams):
    assert (B.gemm_route(B.GEMM_NT, epilogue, G, M, N, K) >= 16) == streams


def test_private_columns_alone_take_the_kernel_of_the_whole_shard():
    """reduce_in_gemm computes the private columns by themselves; their bits are those of the default path, so the order of
    the sums has to be: one sum (tiles) or one per wave (streaming)."""
    for M in (65, 100, 128):
        for G, h, K in ((8, 2048, 264), (8, 4096, 1376), (4, 4096, 512), (2, 2048, 1032), (8, 1024, 4096)):
            whole = B.gemm_route(B.GEMM_NT, ROWPAR, G, M, h, K) >= 16
            for part in range(8, h, 8):
                assert (B.gemm_route(B.GEMM_NT, ROWPAR, G, M, part, K, 1, h) >= 16) == whole


SHARED = 6


@pytest.mark.parametrize("M,N,K,T,best", [(777, 2048, 1376, 8, (4, 8)), (65, 2048, 512, 8, (4, 8)), (777, 2048, 3584, 4, (4,)),
                                          (777, 1024, 512, 4, (1,)), (1024, 1024, 512, 4, (1,)), (2048, 512, 512, 4, (1,))])
def test_shared_channels_are_cut_into_groups_of_ranks_where_that_is_faster(M, N, K, T, best):
    assert max(B.gemm_route(B.GEMM_NT, SHARED, 1, M, N, K, T) // 256, 1) in best


# ---------------------------------------------------------------- what the GPU tests reach
GELU_BWD, SWIGLU_BWD = 4, 5


def _route(layout, epilogue, *sizes):
    r = B.gemm_route(layout, epilogue, *sizes)
    return layout, epilogue, r if r < 256 else 256 + r % 256      # the number of groups of ranks does not matter


def _mlp_gemms(swi, T, n, h, fr, hs, reduce_in_gemm):
    """The GEMM launches of an MLP block, forward and backward."""
    pw = 2 * fr if swi else fr
    out = [(B.GEMM_NT, SWIGLU if swi else GELU, T, n, fr, h)]
    if reduce_in_gemm and n > 64 and hs % 8 == 0:
        out += [(B.GEMM_NT, ROWPAR, T, n, h - hs, fr, 1, h)] * (hs < h) + [(B.GEMM_NT, SHARED, 1, n, hs, fr, T)] * (hs > 0)
    else:
        out.append((B.GEMM_NT, ROWPAR, T, n, h, fr))
    return out + [(B.GEMM_NN, SWIGLU_BWD if swi else GELU_BWD, T, n, fr, h), (B.GEMM_TN, PLAIN, T, h, fr, n),
                  (B.GEMM_NN, PLAIN, T, n, h, pw), (B.GEMM_TN, PLAIN, T, pw, h, n)]


def _reachable():
    rows = (1, 16, 17, 33, 48, 49, 65, 100, 128, 136, 200, 456, 777, 1000, 1300, 2048)
    cols = (8, 72, 136, 520, 1032, 1160, 1544, 2056, 3080, 4104, 6152)
    depths = (8, 72, 264, 1032, 1160, 3080)
    for G in (1, 2, 4, 8, 16):
        for M in rows:
            for N in cols:
                for K in depths:
                    yield from ((B.GEMM_NT, e, G, M, N, K) for e in (PLAIN, GELU, SWIGLU, ROWPAR))
                    yield from ((B.GEMM_NN, e, G, M, N, K) for e in (PLAIN, GELU_BWD, SWIGLU_BWD))
                    if M % 8 == 0:
                        yield B.GEMM_TN, PLAIN, G, M, N, K
                    if M > 64 and G > 1:
                        yield B.GEMM_NT, SHARED, 1, M, N, K, G


def test_exact_gemm_tests_walk_over_several_large_tiles():
    """The persistent tiles (0 to 2) with more tiles than compute units, 1, 2 and 3 stages of k or 2 and 3, in every layout."""
    from tests import test_gpu_gemm_exact as exact
    size = {0: (256, 256), 1: (192, 256), 2: (256, 192)}
    walks = set()
    for layout in (B.GEMM_NT, B.GEMM_NN, B.GEMM_TN):
        for G, M, N, K in exact.SHAPES:
            r = B.gemm_route(layout, PLAIN, G, M, N, K)
            if r in size and G * -(-M // size[r][0]) * -(-N // size[r][1]) > 256:
                walks.add((layout, r, -(-K // 64)))
        assert {(layout, 0, s) for s in (1, 2, 3)} | {(layout, r, s) for r in (1, 2) for s in (2, 3)} <= walks


def test_gpu_tests_reach_every_gemm_kernel():
    from tests import test_gpu_gemm_exact as exact
    from tests import test_gpu_gemm_kernels as blocks
    covered = {_route(*g) for b in blocks.BLOCKS for g in _mlp_gemms(*b)}
    covered |= {_route(layout, PLAIN, *s) for s in exact.SHAPES for layout in (B.GEMM_NT, B.GEMM_NN, B.GEMM_TN)}
    covered |= {_route(B.GEMM_NT, PLAIN, G, M, N, K) for G, N, K in exact.FEW_ROWS for M in exact.FEW_ROWS_M}
    missing = {_route(*g) for g in _reachable()} - covered
    assert not missing, sorted(missing)
