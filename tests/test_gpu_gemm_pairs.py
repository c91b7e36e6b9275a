"""The backward's GEMMs two to a launch: every tile shape with every fused epilogue that a pair has, and the same launches one
after the other, which the library takes while launches are timed."""
import numpy as np
import pytest

from paper_2506_19645_amd import binding as B
from tests.test_gpu_block import check_mlp_block, oracle_mlp_block, run_mlp_block
from tests.test_gpu_gemm_kernels import BLOCKS, block_config
from tests.util import make_inputs

pytestmark = pytest.mark.gpu

# (SwiGLU, T, tokens, h, ffn / T, hs); contractions with a remainder, ragged edges, more tiles than the chip holds at once and
# fewer; tests/test_gemm_pair_routes.py checks on the host which launches they reach
PAIRS = [
    (False, 8, 1000, 1032, 520, 512), (True, 8, 1000, 1032, 520, 21), (False, 4, 1300, 1160, 1032, 0), (True, 4, 1300, 1160, 1032, 1160),
    (False, 8, 136, 264, 2056, 64), (True, 8, 136, 264, 2056, 79), (True, 8, 1160, 264, 1032, 264), (False, 2, 1300, 1032, 1544, 512),
    (True, 2, 1300, 1032, 1544, 0), (False, 16, 1300, 1032, 136, 512), (True, 4, 200, 1160, 4104, 256), (False, 8, 136, 1160, 2056, 576),
    (False, 8, 1, 72, 3080, 40), (True, 16, 1, 72, 1544, 72), (False, 8, 100, 8, 3080, 8), (True, 16, 100, 72, 1544, 0),
    (False, 4, 65, 8, 3080, 0), (True, 8, 65, 136, 1544, 100), (False, 4, 1, 136, 2056, 136), (True, 8, 17, 72, 1032, 21),
    (False, 1, 1, 8, 8, 4), (True, 2, 65, 72, 136, 33), (False, 2, 100, 136, 200, 64), (True, 2, 33, 200, 72, 128),
    (False, 2, 256, 768, 1536, 384), (False, 2, 2048, 1032, 3080, 0), (True, 4, 1300, 264, 2056, 128),
    (False, 4, 1300, 264, 4104, 128), (True, 1, 65, 8, 72, 5), (True, 4, 100, 72, 1544, 32), (True, 8, 65, 72, 1032, 72), (True, 8, 100, 8, 2056, 8),
    # persistent tiles walked several to a workgroup: by the first GEMM and, in shares, by the second, either one the data
    # gradient, with ragged edges; the GELU and the SwiGLU derivative among those that walk
    (True, 8, 264, 1672, 488, 837), (True, 16, 136, 1288, 72, 640), (True, 16, 264, 136, 2056, 72), (False, 16, 264, 136, 2056, 21),
    (True, 16, 456, 2192, 200, 1096), (True, 16, 390, 2056, 72, 513), (True, 16, 777, 1288, 264, 0), (True, 16, 264, 2072, 72, 2072),
    (True, 16, 390, 2184, 200, 546), (True, 16, 390, 1288, 264, 648), (True, 16, 264, 2056, 264, 100), (True, 16, 136, 1800, 264, 904),
]

# (T, tokens, h, ffn / T, hs): private and shared columns of a product with the reduce inside in one launch, summed in groups of
# ranks and directly
SHARED = [
    (8, 456, 3080, 72, 8), (8, 136, 4096, 264, 8), (2, 1300, 3080, 72, 8), (8, 200, 3080, 72, 8), (8, 777, 1032, 72, 8), (8, 65, 2056, 264, 8),
    (4, 136, 72, 264, 32), (8, 2048, 4096, 72, 2048), (8, 1300, 3080, 72, 8), (4, 1300, 2056, 1032, 1024), (2, 456, 4096, 8, 8),
    (2, 1000, 2056, 72, 1024), (8, 456, 2056, 264, 1024), (2, 200, 4096, 8, 8), (8, 65, 4096, 264, 4088), (2, 136, 72, 8, 32),
    (8, 65, 2056, 264, 2048),
    # stored to all ranks from the pair itself; several persistent tiles to a workgroup: private columns first, either part second in shares
    (2, 3500, 3352, 1072, 2448), (2, 2056, 4056, 416, 3984), (2, 1160, 3440, 8, 3408), (16, 264, 3248, 72, 8), (16, 390, 1088, 88, 16),
    (16, 264, 4136, 72, 400), (8, 2056, 944, 656, 544),
]


def paired(swi, T, n, h, fr):
    """Whether any of a backward pass's pairs of GEMMs shares a launch."""
    return B.gemm_pair_route(T, n, fr, h) >= 0 or B.gemm_pair_route(T, n, h, 2 * fr if swi else fr) >= 0


def check(swi, T, n, h, fr, hs):
    cfg = block_config(swi, T, n, h, fr, hs)
    d = make_inputs(cfg, seed=31, weight_std=0.05)
    got = run_mlp_block(cfg, d)
    w, fwd, g = oracle_mlp_block(cfg, d)
    check_mlp_block(cfg, d, got, w, fwd, g)


@pytest.mark.parametrize("swi,T,n,h,fr,hs", PAIRS)
def test_mlp_block_with_paired_gemms(swi, T, n, h, fr, hs):
    check(swi, T, n, h, fr, hs)


@pytest.mark.parametrize("swi,T,n,h,fr,hs", [b[:6] for b in BLOCKS])
def test_mlp_block_with_every_gemm_a_launch_of_its_own(swi, T, n, h, fr, hs):
    if not paired(swi, T, n, h, fr):
        pytest.skip("two launches anyway, as tests/test_gpu_gemm_kernels.py runs them")
    B.profile_reset()
    B.profile_enable(True)
    try:
        check(swi, T, n, h, fr, hs)
    finally:
        B.profile_enable(False)
    assert sum(name.startswith("gemm") for name, _ in B.profile_records()) == 6
    B.profile_reset()


@pytest.mark.parametrize("T,n,h,fr,hs", SHARED)
def test_reduce_in_gemm_with_both_parts_in_one_launch(T, n, h, fr, hs):
    cfg = block_config(False, T, n, h, fr, hs)
    d = make_inputs(cfg, seed=37, weight_std=0.05)
    got = run_mlp_block(cfg, d, reduce_in_gemm=True)
    w, fwd, g = oracle_mlp_block(cfg, d)
    check_mlp_block(cfg, d, got, w, fwd, g)
    other = run_mlp_block(cfg, d, backward=False)
    assert np.array_equal(got["Rp_bits"][:, :, hs:], other["Rp_bits"][:, :, hs:])   # private channels: the same bits
    B.profile_reset()
    B.profile_enable(True)
    try:
        two = run_mlp_block(cfg, d, backward=False, reduce_in_gemm=True)            # the two parts one after the other
    finally:
        B.profile_enable(False)
        B.profile_reset()
    assert np.array_equal(got["Rp_bits"], two["Rp_bits"])                           # all channels: the same bits
