"""A number of shared channels that ends inside a 16-byte group: the kernels that reduce and normalise in one launch against the
two kernels (the residual: the same bits) and the oracle; the stand-alone entry point still refuses it."""
import numpy as np
import pytest

from paper_2506_19645_amd import binding as B
from paper_2506_19645_amd import inputs as I
from tests.test_gpu_block import check_mlp_block, oracle_mlp_block, run_mlp_block
from tests.test_gpu_decode import oracle_decode, run_decode
from tests.util import assert_close, make_inputs, ulp_distance_bf16

pytestmark = pytest.mark.gpu


def cfg_of(swi, T, n, h, hs, scale=1.0):
    return I.BlockConfig("k", I.KIND_MLP_SWIGLU if swi else I.KIND_MLP_GELU, I.NORM_RMSNORM if swi else I.NORM_LAYERNORM, h=h, T=T,
                         p=(hs + 0.5) / h, batch=1, seq=n, ffn=T * 72, private_scale=scale)


@pytest.mark.parametrize("swi,T,n,h,hs,scale", [
    (False, 2, 1, 8, 1, 1.0), (True, 2, 300, 72, 71, 1.5), (False, 2, 33, 2056, 2049, 2.0), (True, 2, 7, 4096, 1435, 1.0),
    (False, 4, 65, 136, 5, 2.0), (True, 4, 257, 2048, 1433, 2.0), (False, 4, 9, 4104, 4100, 1.0), (True, 8, 40, 1032, 517, 1.0),
    (False, 8, 3, 8192, 8190, 1.0), (True, 16, 17, 520, 3, 4.0), (False, 16, 2, 4096, 2047, 1.0),
    # two tokens at a time in the backward: ranges of 2, 3 and 4 tokens, the last one shorter
    (False, 4, 1111, 768, 381, 2.0), (True, 2, 1537, 1024, 512, 1.0), (False, 2, 2049, 1024, 1000, 1.5), (True, 4, 600, 520, 519, 1.0),
    # up to 512 channels the backward keeps two kernels from 3000 tokens on (RMSNorm: among so many values LayerNorm's beta leaves
    # some near zero, whose bf16 steps are smaller than what the statistics' last bit moves them by)
    (True, 4, 2999, 512, 253, 1.0), (True, 4, 3000, 512, 253, 1.0), (True, 2, 3000, 264, 256, 1.5), (True, 2, 3000, 520, 513, 1.0)])
def test_mlp_block_with_a_ragged_number_of_shared_channels(swi, T, n, h, hs, scale):
    cfg = cfg_of(swi, T, n, h, hs, scale)
    d = make_inputs(cfg, seed=43, weight_std=0.05 if h < 4096 else 0.02)
    got = run_mlp_block(cfg, d)
    w, fwd, g = oracle_mlp_block(cfg, d)
    check_mlp_block(cfg, d, got, w, fwd, g)
    two = run_mlp_block(cfg, d, separate_reduce=True)
    assert np.array_equal(got["Rp_bits"], two["Rp_bits"])
    # a row's squares are added up in another order: statistics to fp32 rounding, normalised values to one bf16 step
    assert ulp_distance_bf16(got["Xp_bits"], two["Xp_bits"]).max() <= 1
    for m in range(1, T):                     # the reduced gradient: the same bits on every rank's shared channels
        assert np.array_equal(got["dZt"][m, :, :hs], got["dZt"][0, :, :hs])
    B.profile_reset()
    B.profile_enable(True)
    try:
        run_mlp_block(cfg, d)
    finally:
        B.profile_enable(False)
    names = {name for name, _ in B.profile_records()}
    assert "partial_sync_norm_fwd" in names and ("norm_bwd_sync" in names) == (T * -(-h // 2048) <= 4 and (h > 512 or n < 3000))
    B.profile_reset()


@pytest.mark.parametrize("T,batch,heads,p", [(2, 1, 16, 0.301), (4, 5, 16, 0.777), (8, 3, 32, 0.5 + 3 / 4096), (8, 300, 16, 0.333), (8, 40, 8, 0.9)])
def test_decode_layer_with_a_ragged_number_of_shared_channels(T, batch, heads, p):
    cfg = I.BlockConfig("d", I.KIND_DECODE, I.NORM_RMSNORM, h=heads * 128, T=T, p=p, batch=batch, seq=1, ffn=T * 136, n_heads=heads,
                        head_dim=128, kv_len=70)
    d = make_inputs(cfg, seed=44, weight_std=0.02)
    one, two = run_decode(cfg, d), run_decode(cfg, d, separate_reduce=True)
    assert np.array_equal(one["R1_bits"], two["R1_bits"])
    ref = oracle_decode(cfg, d)
    for name in ("R1", "X2", "R2"):
        assert_close(one[name], ref[name], name)


def test_the_stand_alone_call_refuses_a_ragged_number():
    import torch
    t = [torch.zeros(2, 4, 64, dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    gamma, rstd = torch.ones(64, dtype=torch.bfloat16, device="cuda"), torch.empty(2, 4, dtype=torch.float32, device="cuda")
    p = B._ptr
    for hs, status in ((12, 6), (0, 6), (16, 0)):
        assert B.lib().caat_partial_sync_norm_fwd(p(t[0]), p(t[1]), p(gamma), None, p(t[2]), None, p(rstd), B.RMSNORM, 2, 4, 64, hs, 1e-5,
                                                  None) == status
    torch.cuda.synchronize()
