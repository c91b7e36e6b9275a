"""Shard GEMM on small integers: every product and sum is exact in fp32 and the result is an integer of at most 8 bits
(|sum| <= 256) or is rounded once to bf16, so the GPU bits must equal the correctly rounded integer result -- at the
edges of the tiles, of the k stages and of the walk over several tiles per workgroup."""
import numpy as np
import pytest

from paper_2506_19645_amd import binding as B
from paper_2506_19645_amd import inputs as I

pytestmark = pytest.mark.gpu

# (G, M, N, K): below / at / past one tile in each dimension; 1, 2 and 3 stages of k with and without a remainder;
# more tiles than compute units with stage counts 1, 2, 3 (the stream of copies runs on from tile to tile).  The tiles named
# below are those of the layouts' choice on 256 compute units; tests/test_gemm_routes.py checks that none is left out
SHAPES = [(1, 8, 8, 8), (2, 256, 256, 64), (1, 264, 248, 72), (1, 520, 776, 200), (3, 296, 520, 136), (1, 24, 136, 320),
          (5, 2048, 2048, 64), (5, 2040, 1928, 128), (5, 2008, 2056, 184),
          # 192 x 256 and 256 x 192 tiles: one round with a remainder in both directions, several tiles per workgroup with
          # 2 and 3 stages; 64 x 128 tiles of 64 rows and a remainder
          (8, 1032, 1160, 200), (8, 1144, 1808, 136), (8, 1000, 1160, 328), (8, 2024, 2200, 72), (8, 2008, 2096, 136),
          (8, 200, 1160, 136),
          # two groups of waves on one contraction, 64 x 64 and 128 x 128 tiles: last stages that one group has to itself
          # and that both share
          (4, 296, 520, 2056), (4, 200, 520, 1096), (8, 456, 776, 1096), (8, 456, 776, 3080),
          # 256 x 256 tiles: one round, and several tiles per workgroup with 1, 2 and 3 stages
          (8, 200, 6152, 72), (5, 1016, 5112, 64), (5, 1016, 5112, 72), (5, 1016, 5112, 136)]


@pytest.mark.parametrize("G,M,N,K", SHAPES)
@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
def test_gemm_small_integers_bit_exact(layout, G, M, N, K):
    import torch
    rng = np.random.default_rng(M * 7 + N * 3 + K + layout)
    a = rng.integers(-2, 3, size=(G, M, K)).astype(np.float32)
    b = rng.integers(-2, 3, size=(G, N, K)).astype(np.float32)
    want = I.f32_to_bf16_bits(np.matmul(a, b.transpose(0, 2, 1)))        # |sum| < 2^24: exact in fp32
    at = a.transpose(0, 2, 1) if layout == B.GEMM_TN else a
    bt = b if layout == B.GEMM_NT else b.transpose(0, 2, 1)
    da, db = B.to_device(I.f32_to_bf16_bits(at)), B.to_device(I.f32_to_bf16_bits(bt))
    out = torch.full((G, M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.gemm_bf16(da, db, out, layout, G, M, N, K, M if layout == B.GEMM_TN else K, K if layout == B.GEMM_NT else N, N,
                M * K, N * K, M * N)
    torch.cuda.synchronize()
    assert np.array_equal(B.to_host_bits(out), want)


# few token rows: one, around 16-row tiles, past 64 and up to the streaming kernel's limit; short and ragged contractions;
# shards whose widths leave a remainder in every tile width; the last two have so many weight rows that more than 16
# token rows take the tile kernel
FEW_ROWS = [(2, 8, 8), (8, 1376, 512), (3, 520, 72), (2, 1288, 2048), (1, 40, 4104), (4, 8192, 136), (16, 2056, 200),
            (2, 4104, 1160), (2, 6152, 1160)]
FEW_ROWS_M = (1, 2, 15, 16, 17, 32, 33, 48, 63, 64, 65, 80, 97, 128, 129)


@pytest.mark.parametrize("G,N,K", FEW_ROWS)
def test_gemm_few_rows_small_integers_bit_exact(G, N, K):
    import torch
    rng = np.random.default_rng(N + K)
    b = rng.integers(-2, 3, size=(G, N, K)).astype(np.float32)
    db = B.to_device(I.f32_to_bf16_bits(b))
    for M in FEW_ROWS_M:
        a = rng.integers(-2, 3, size=(G, M, K)).astype(np.float32)
        want = I.f32_to_bf16_bits(np.matmul(a, b.transpose(0, 2, 1)))
        da = B.to_device(I.f32_to_bf16_bits(a))
        out = torch.full((G, M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        B.gemm_bf16(da, db, out, B.GEMM_NT, G, M, N, K, K, K, N, M * K, N * K, M * N)
        torch.cuda.synchronize()
        assert np.array_equal(B.to_host_bits(out), want), M
