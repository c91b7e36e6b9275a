"""q and k rotated in the epilogue of the product that makes them, and k and v stored to the caches there: every tile that can,
sequences that end in and between a wave's 16-row steps, against the pass of its own and the oracle."""
import numpy as np
import pytest

from paper_2506_19645_amd import binding as B
from paper_2506_19645_amd import inputs as I
from tests.test_gpu_attn import _cfg as attn_cfg, check_attn, oracle_attn_block, run_attn_block
from tests.test_gpu_decode import run_decode
from tests.test_gpu_prefill import _cfg as prefill_cfg, check_prefill, oracle_prefill, run_prefill
from tests.util import assert_close, bits_to_f64, make_inputs

pytestmark = pytest.mark.gpu

# T, heads, key heads, sequences, tokens, base; the tile of the product
CASES = [(2, 4, 4, 400, 7, 1e4, 3), (2, 4, 2, 130, 16, 1e4, 4), (2, 2, 2, 3, 1003, 1e4, 4), (1, 8, 2, 5, 333, 5e5, 4),
         (2, 8, 8, 9, 257, 1e4, 3), (4, 8, 4, 31, 65, 0.5, 4), (2, 8, 2, 300, 17, 1e4, 3), (1, 4, 4, 1, 2049, 1e4, 4),
         (4, 8, 8, 200, 33, 1e4, 1), (4, 8, 8, 310, 32, 1e4, 0), (4, 8, 8, 23, 431, 1.5, 0)]


def timed(run):
    """The same with every launch timed, where the rotation is a pass of its own."""
    B.profile_reset()
    B.profile_enable(True)
    try:
        return run(), {name for name, _ in B.profile_records()}
    finally:
        B.profile_enable(False)
        B.profile_reset()


def check_rotated(a, b, dh=128):
    """Heads [..., 128] rotated on two routes: each rounds to bf16 (to half a step, at most 2^-8 of the value: one step apart).  The
    angles are the same; the sines and cosines are the hardware's, each good to 2.6e-7, directly on one route and on the other
    turned on up to eight times by those of 16 positions (10 x sqrt(2) x 2.6e-7, and 8 x 3 roundings of 2^-24: 5.1e-6)."""
    a, b = (x.reshape(x.shape[:-1] + (-1, 2, dh // 2)) for x in (a, b))
    size = np.sqrt((b ** 2).sum(axis=-2, keepdims=True))
    assert (np.abs(a - b) <= 2.0 ** -7 * np.maximum(np.abs(a), np.abs(b)) + 8e-6 * size).all()


@pytest.mark.parametrize("T,heads,kv,batch,seq,base,tile", CASES)
def test_attention_block(T, heads, kv, batch, seq, base, tile):
    cfg = attn_cfg(T, batch, seq, heads, 0.5, kv_heads=kv).with_(rope_base=base)
    assert B.gemm_route(B.GEMM_NT, 0, T, cfg.tokens, cfg.qkv_r, cfg.h) == tile
    d = make_inputs(cfg, seed=47, with_grads=False, weight_std=0.05 if cfg.h < 1024 else 0.02)
    got = run_attn_block(cfg, d)
    two, names = timed(lambda: run_attn_block(cfg, d))
    assert "rope" in names
    rot = cfg.hd_r + cfg.kvd_r
    check_rotated(got["QKV"][..., :rot], two["QKV"][..., :rot])
    assert np.array_equal(got["QKV"][..., rot:], two["QKV"][..., rot:])
    check_attn(cfg, d, got, oracle_attn_block(cfg, d)[1])


@pytest.mark.parametrize("T,heads,kv,batch,seq,base,tile", CASES)
def test_prefill_layer(T, heads, kv, batch, seq, base, tile):
    cfg = prefill_cfg(T, batch, seq, heads, T * 136, 0.5, kv_heads=kv).with_(rope_base=base)
    assert B.gemm_route(B.GEMM_NT, 0, T, cfg.tokens, cfg.qkv_r, cfg.h) == tile
    d = make_inputs(cfg, seed=48, weight_std=0.05 if cfg.h < 1024 else 0.02)
    got = run_prefill(cfg, d, kv_cap=seq + 5)
    two, names = timed(lambda: run_prefill(cfg, d, kv_cap=seq + 5))
    assert "rope_kv_append" in names
    k, v = got["Kc_bits"], got["Vc_bits"]
    assert not k[:, :, :, seq:].any() and not v[:, :, :, seq:].any()
    check_rotated(bits_to_f64(k[:, :, :, :seq]), bits_to_f64(two["Kc_bits"][:, :, :, :seq]))
    assert np.array_equal(v, two["Vc_bits"])
    w, ref = oracle_prefill(cfg, d)
    check_prefill(cfg, d, got, ref)
    assert_close(bits_to_f64(k[:, :, :, :seq]), ref["K"], "K cache")
    assert_close(bits_to_f64(v[:, :, :, :seq]), ref["V"], "V cache")


@pytest.mark.parametrize("batch,seq", [(9921, 1), (1417, 7), (1240, 8)])
def test_short_sequences_on_large_tiles(batch, seq):
    """From 8 tokens on in the epilogue of a 256 x 256 tile; the pass and the epilogue agree."""
    cfg = attn_cfg(4, batch, seq, 8, 0.5)
    assert B.gemm_route(B.GEMM_NT, 0, 4, cfg.tokens, cfg.qkv_r, cfg.h) == 0
    d = make_inputs(cfg, seed=52, with_grads=False)
    B.profile_reset()
    B.profile_enable(True, as_run=True)
    try:
        got = run_attn_block(cfg, d)
        names = {name for name, _ in B.profile_records()}
    finally:
        B.profile_enable(False)
        B.profile_reset()
    assert ("rope" in names) == (seq < 8)
    two, _ = timed(lambda: run_attn_block(cfg, d))
    rot = cfg.hd_r + cfg.kvd_r
    check_rotated(got["QKV"][..., :rot], two["QKV"][..., :rot])
    assert np.array_equal(got["QKV"][..., rot:], two["QKV"][..., rot:])


# far out in a sequence, where an angle of a position times an fp32 frequency that is rounded once is off by 1e-3
FAR = 20000


def one_hot(cfg, d):
    """Projections that pick a channel each, so that q, k and v have the same bits whatever kernel makes them."""
    w = np.zeros_like(d["Wqkv"])
    w[0, np.arange(cfg.qkv_r), np.random.default_rng(7).integers(0, cfg.h, cfg.qkv_r)] = 0x3F80
    return dict(d, Wqkv=w)


def test_far_positions_in_prefill_and_decode():
    """The key that a decode step appends at position 20000, and that a prompt of that length has there, rotated in the product's
    epilogue and as a pass of its own."""
    cfg = prefill_cfg(1, 1, FAR + 1, 4, 136, 0.0)
    assert B.gemm_route(B.GEMM_NT, 0, 1, cfg.tokens, cfg.qkv_r, cfg.h) in (0, 1, 3, 4)
    d = one_hot(cfg, make_inputs(cfg, seed=49, weight_std=0.05))
    # a sum of squares that is exact in any order, so the norm kernels agree too
    d["R"] = np.random.default_rng(8).choice(np.array([0x3F00, 0x3F80, 0x4000, 0xBF00, 0xBF80, 0xC000], dtype=np.uint16), d["R"].shape)
    d["gamma_attn"][:] = 0x3F80
    one = run_prefill(cfg, d, kv_cap=FAR + 1)["Kc_bits"]
    two, names = timed(lambda: run_prefill(cfg, d, kv_cap=FAR + 1)["Kc_bits"])
    assert "rope_kv_append" in names
    check_rotated(bits_to_f64(one), bits_to_f64(two))
    step = I.BlockConfig("d", I.KIND_DECODE, I.NORM_RMSNORM, h=cfg.h, T=1, p=0.0, batch=1, seq=1, ffn=136, n_heads=4, head_dim=128, kv_len=FAR)
    sd = dict(make_inputs(step, seed=50, weight_std=0.05), R=np.ascontiguousarray(d["R"][:, -1:]), Wqkv=d["Wqkv"], gamma_attn=d["gamma_attn"])
    new = run_decode(step, sd)["Kc_bits"][:, :, :, FAR]
    check_rotated(bits_to_f64(new), bits_to_f64(two[:, :, :, FAR]))
    check_rotated(bits_to_f64(new), bits_to_f64(one[:, :, :, FAR]))


def test_far_positions_in_the_attention_block():
    cfg = attn_cfg(1, 1, FAR + 1, 4, 0.0)
    d = one_hot(cfg, make_inputs(cfg, seed=51, with_grads=False))
    one = run_attn_block(cfg, d)["QKV"]
    two, names = timed(lambda: run_attn_block(cfg, d)["QKV"])
    assert "rope" in names
    check_rotated(one[..., :2 * cfg.hd_r], two[..., :2 * cfg.hd_r])
