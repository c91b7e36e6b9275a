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
    (SWIGLU, 4, 3584, 4096, 48, True), (ROWPAR, 8, 4096, 1376, 48, False), (ROWPAR, 8, 4096, 1376, 16, True),
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
