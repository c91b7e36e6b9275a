"""Every kernel that a shard GEMM can be sent to, with every fused epilogue it has, in MLP blocks against the oracle.  All
contractions have more than one stage of k and a remainder, most launches ragged edges, and hs lies inside a tile."""
import pytest

from paper_2506_19645_amd import inputs as I
from tests.test_gpu_block import check_mlp_block, oracle_mlp_block, run_mlp_block
from tests.util import make_inputs

pytestmark = pytest.mark.gpu

# (SwiGLU, T, tokens, h, ffn / T, hs, reduce in the GEMM); tests/test_gemm_routes.py checks on the host that they reach
# every kernel that sizes like these can reach
BLOCKS = [
    (True, 8, 1, 72, 1736, 32, False), (True, 8, 16, 136, 1200, 64, False), (False, 8, 40, 72, 2040, 32, False),
    (False, 8, 33, 2040, 72, 1000, False),
    (True, 1, 1, 200, 72, 60, False), (False, 1, 1, 72, 1160, 16, False), (False, 4, 1, 3080, 72, 1536, True),
    (False, 6, 1, 72, 2056, 16, False), (False, 8, 5, 1160, 1160, 576, True), (False, 8, 5, 1544, 1544, 0, False),
    (True, 8, 17, 1032, 72, 1032, True), (True, 2, 17, 72, 2056, 32, True), (False, 8, 17, 72, 1032, 16, False),
    (True, 16, 17, 72, 520, 72, True), (False, 2, 17, 6152, 72, 6152, False), (False, 3, 17, 72, 4104, 0, False),
    (True, 4, 17, 72, 4104, 21, False), (False, 6, 49, 4104, 72, 1024, False), (False, 6, 49, 72, 4104, 32, False),
    (True, 16, 65, 520, 136, 256, False), (False, 2, 65, 72, 2056, 32, True), (True, 1, 65, 72, 4104, 21, False),
    (False, 4, 65, 72, 2056, 16, True), (True, 1, 77, 4104, 72, 2048, False), (False, 8, 96, 72, 72, 32, True),
    (True, 1, 100, 72, 72, 32, True), (True, 16, 100, 520, 136, 520, False), (False, 1, 100, 6152, 72, 1536, False),
    (True, 8, 100, 72, 520, 32, False), (False, 3, 100, 72, 1544, 32, True), (False, 1, 100, 72, 6152, 72, True),
    (False, 4, 100, 72, 2056, 32, False), (False, 1, 128, 4104, 72, 2048, False), (True, 8, 129, 72, 4104, 32, False),
    (False, 8, 131, 72, 4104, 16, True), (True, 4, 200, 72, 4104, 32, True), (False, 1, 456, 4104, 72, 4104, True),
    (False, 16, 456, 2056, 328, 2056, True), (False, 16, 570, 1800, 328, 1800, True), (False, 8, 777, 328, 520, 328, True),
    (False, 8, 777, 1160, 264, 576, False), (False, 6, 777, 72, 2056, 16, True), (True, 16, 777, 72, 520, 21, False),
    (False, 8, 777, 584, 584, 584, True), (True, 4, 777, 72, 3080, 16, False), (False, 16, 1111, 72, 72, 16, False),
    (True, 16, 1111, 136, 72, 32, False), (False, 16, 1300, 264, 264, 79, False), (False, 1, 1300, 6152, 72, 6152, True),
    (False, 1, 2047, 2056, 136, 2056, True), (True, 6, 2047, 1032, 200, 0, False), (True, 2, 2047, 6152, 72, 6152, True),
    (False, 3, 2047, 5128, 72, 5128, True), (False, 8, 900, 3080, 712, 3080, True),
]


def block_config(swi, T, n, h, fr, hs):
    p = 1.0 if hs == h else (hs + 0.5) / h          # floor(h p) = hs
    return I.BlockConfig("k", I.KIND_MLP_SWIGLU if swi else I.KIND_MLP_GELU, I.NORM_RMSNORM if swi else I.NORM_LAYERNORM, h=h, T=T,
                         p=p, batch=1, seq=n, ffn=T * fr)


@pytest.mark.parametrize("swi,T,n,h,fr,hs,reduce_in_gemm", BLOCKS)
def test_mlp_block_on_every_gemm_kernel(swi, T, n, h, fr, hs, reduce_in_gemm):
    cfg = block_config(swi, T, n, h, fr, hs)
    d = make_inputs(cfg, seed=29, weight_std=0.05)
    got = run_mlp_block(cfg, d, reduce_in_gemm=reduce_in_gemm)
    w, fwd, g = oracle_mlp_block(cfg, d)
    check_mlp_block(cfg, d, got, w, fwd, g)
