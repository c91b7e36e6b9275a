"""GPU parity of the decode layer (one new token per sequence over a KV cache) against the CPU oracle."""
import numpy as np
import pytest

from oracle import caat_oracle as O
from paper_2506_19645_amd import binding as B
from paper_2506_19645_amd import inputs as I
from tests.util import assert_close, bits_to_f64, make_inputs, hs_of

pytestmark = pytest.mark.gpu


def run_decode(cfg, d, reduce_in_gemm=False, separate_reduce=False, ws=None):
    import torch
    desc = B.make_desc(cfg, reduce_in_gemm=reduce_in_gemm, separate_reduce=separate_reduce)
    T, b, h, hd = cfg.T, cfg.batch, cfg.h, cfg.hd_r
    weights = [B.to_device(d["gamma_attn"]), B.to_device(d["Wqkv"]), B.to_device(d["Wo"]), B.to_device(d["gamma"]),
               B.to_device(np.concatenate([d["Wg"], d["Wu"]], axis=1)), B.to_device(d["B"])]
    r = B.to_device(d["R"])
    kc, vc = B.to_device(d["Kc"]), B.to_device(d["Vc"])
    r_out = torch.empty_like(r)
    if ws is None:
        ws = torch.zeros(B.workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    B.block_fwd(desc, weights, None, r, r_out, None, ws, kv_k=kc, kv_v=vc)
    torch.cuda.synchronize()
    L = B.workspace_layout(desc)

    def ws_bf16(off, nbytes, shape):
        return bits_to_f64(ws[off:off + nbytes].view(torch.int16).cpu().numpy().view(np.uint16).reshape(shape))

    return {"R2": bits_to_f64(B.to_host_bits(r_out)), "R2_bits": B.to_host_bits(r_out),
            "X1": ws_bf16(L.off_X1, L.bytes_X1, (T, b, h)), "H": ws_bf16(L.off_H, L.bytes_H, (T, b, hd)),
            "R1": ws_bf16(L.off_R1, L.bytes_R1, (T, b, h)), "X2": ws_bf16(L.off_X2, L.bytes_X2, (T, b, h)),
            "R1_bits": ws[L.off_R1:L.off_R1 + L.bytes_R1].view(torch.int16).cpu().numpy().view(np.uint16).reshape(T, b, h),
            "Kc_bits": B.to_host_bits(kc), "Vc_bits": B.to_host_bits(vc)}


def _cfg(T, b, heads, ffn, L, p, kv_heads=0, scale=1.0):
    return I.BlockConfig("dec", I.KIND_DECODE, I.NORM_RMSNORM, h=heads * 128, T=T, p=p, batch=b, seq=1, ffn=ffn,
                         n_heads=heads, head_dim=128, kv_len=L, n_kv_heads=kv_heads, private_scale=scale)


def oracle_decode(cfg, d):
    w = {k: O.widen_bf16(v) for k, v in d.items()}
    return O.decode_layer_fwd(w["R"], w, w["Kc"], w["Vc"], kv_len=cfg.kv_len, heads_per_rank=cfg.n_heads // cfg.T,
                              head_dim=cfg.head_dim, hs=hs_of(cfg), eps=cfg.eps, private_scale=cfg.private_scale,
                              rope_base=cfg.rope_base, kv_heads_per_rank=cfg.kv_heads // cfg.T)


@pytest.mark.parametrize("T,b,heads,ffn,L,p,kv_heads,scale", [
    (2, 3, 4, 2 * 344, 37, 0.5, 0, 1.0),      # fewer keys than one 64-key sweep, ragged ffn shard
    (2, 64, 4, 2 * 256, 300, 0.25, 0, 1.0),   # the benchmark's batch, several sweeps + tail
    (4, 5, 4, 4 * 128, 0, 1.0, 0, 1.0),       # empty cache: the token attends to itself only
    (1, 2, 2, 256, 129, 0.0, 0, 1.0),
    (2, 5, 8, 2 * 256, 200, 0.5, 2, 1.0),     # grouped-query attention: 4 query heads per key / value head
    (2, 3, 8, 2 * 256, 70, 0.5, 4, 1.0),      # two groups per rank
    (2, 4, 4, 2 * 256, 50, 0.3, 0, 1.0),      # hs = 153 ends inside a 16-byte group, in the one-launch reduce + norm
    (8, 6, 8, 8 * 128, 90, 0.5, 0, 1.0),      # tensor-parallel degree 8 through the one-launch reduce + norm
    (4, 7, 4, 4 * 128, 61, 0.5, 0, 2.0),      # private channel scaling sqrt(T) (Sec. 4) in both halves of the layer
    (2, 5, 4, 2 * 256, 40, 0.0, 0, 2.0 ** 0.5),   # the same at p = 0: every channel private and scaled
    (16, 3, 32, 16 * 128, 70, 0.5, 0, 1.0),   # tensor-parallel degree 16 (Sec. 5's largest): 32 heads, 2 per rank
    (4, 3, 12, 4 * 128, 40, 0.5, 0, 1.0),     # reduce + norm per token and rank: one column group per thread (h = 1536), ...
    (2, 5, 20, 2 * 256, 30, 0.25, 0, 1.0),    # ... two (2560, the second one ragged), ...
    (8, 2, 40, 8 * 128, 20, 0.4, 8, 1.0),     # ... and four (5120), hs = 2048
    (16, 2, 32, 16 * 136, 20, 0.3, 0, 4.0),   # T = 16, hs not a multiple of 8 (one launch, in place), scaling sqrt(T)
])
def test_decode_layer(T, b, heads, ffn, L, p, kv_heads, scale):
    cfg = _cfg(T, b, heads, ffn, L, p, kv_heads, scale)
    d = make_inputs(cfg, seed=31, weight_std=0.05 if cfg.h < 4096 else 0.02)   # h = 4096: scores stay O(1), as in the benchmark
    got = run_decode(cfg, d)
    ref = oracle_decode(cfg, d)
    assert_close(got["X1"], ref["X1"], "X1")
    assert_close(got["H"], ref["H"], "H")
    assert_close(got["R1"], ref["R1"], "R1")
    assert_close(got["X2"], ref["X2"], "X2")
    assert_close(got["R2"], ref["R2"], "R2")
    # the new token's rotated k and its v were appended at position L; every older cache row keeps its bits
    assert_close(bits_to_f64(got["Kc_bits"][:, :, :, L]), ref["k_new"], "k_new")
    assert_close(bits_to_f64(got["Vc_bits"][:, :, :, L]), ref["v_new"], "v_new")
    assert np.array_equal(got["Kc_bits"][:, :, :, :L], d["Kc"][:, :, :, :L])
    assert np.array_equal(got["Vc_bits"][:, :, :, :L], d["Vc"][:, :, :, :L])
    hs = hs_of(cfg)
    if hs > 0 and T > 1 and np.array_equal(d["R"][0, :, :hs], d["R"][-1, :, :hs]):
        for m in range(1, T):
            assert np.array_equal(got["R2_bits"][m, :, :hs], got["R2_bits"][0, :, :hs])
            assert np.array_equal(got["R1_bits"][m, :, :hs], got["R1_bits"][0, :, :hs])


@pytest.mark.parametrize("T,b,heads,ffn,L,p,scale", [
    (2, 4, 4, 2 * 256, 50, 0.3, 1.0), (16, 2, 32, 16 * 136, 20, 0.3, 4.0), (8, 5, 16, 8 * 72, 33, 0.777, 1.0), (4, 1, 20, 4 * 128, 17, 1.0, 1.0)])
def test_decode_layer_with_the_reduce_and_the_norm_as_two_kernels(T, b, heads, ffn, L, p, scale):
    """The same against the oracle where the caller asks for the reduce as a kernel of its own; hs a multiple of 8 and not."""
    cfg = _cfg(T, b, heads, ffn, L, p, 0, scale)
    d = make_inputs(cfg, seed=34, weight_std=0.05 if cfg.h < 4096 else 0.02)
    B.profile_reset()
    B.profile_enable(True, as_run=True)
    try:
        got = run_decode(cfg, d, separate_reduce=True)
        names = [name for name, _ in B.profile_records()]
    finally:
        B.profile_enable(False)
        B.profile_reset()
    assert names.count("partial_sync_fwd") == 2 and "partial_sync_norm_fwd" not in names
    ref = oracle_decode(cfg, d)
    for name in ("X1", "H", "R1", "X2", "R2"):
        assert_close(got[name], ref[name], name)


@pytest.mark.parametrize("separate", [False, True])
def test_decode_layer_outputs_alone_with_a_tiny_residual(separate):
    """With the residual stream scaled down by 2^-10 (RMSNorm does not care, up to eps) both R1 and R2 are dominated by
    the reduced sub-layer outputs Z, so the relative error is measured against Z itself and not hidden behind
    R ~ N(0,1); run through both routes (one-launch reduce + norm, and the reduce as a kernel of its own)."""
    cfg = _cfg(4, 9, 8, 4 * 256, 150, 0.5)
    d = make_inputs(cfg, seed=33, weight_std=0.05)
    d["R"] = I.f32_to_bf16_bits(I.bf16_bits_to_f32(d["R"]) * np.float32(2.0 ** -10))     # exact: a power of two
    got = run_decode(cfg, d, separate_reduce=separate)
    ref = oracle_decode(cfg, d)
    assert np.abs(ref["R1"] - O.widen_bf16(d["R"])).max() > 50 * np.abs(O.widen_bf16(d["R"])).max()
    for name in ("R1", "X2", "R2"):
        assert_close(got[name], ref[name], name)
    hs = hs_of(cfg)
    for m in range(1, cfg.T):
        assert np.array_equal(got["R2_bits"][m, :, :hs], got["R2_bits"][0, :, :hs])


@pytest.mark.parametrize("T,b,heads,kv_heads,L", [
    (2, 1, 4, 0, 15),        # one block of 16 keys, the new key its last row
    (2, 1, 4, 0, 16),        # the new key opens a block
    (2, 3, 8, 2, 1023),      # few sequences, long cache: many ranges of keys, four query heads per key / value head
    (1, 1, 2, 1, 2050),      # two query heads, 64 ranges at most
    (2, 2, 34, 2, 333),      # 17 query heads per key / value head: a second workgroup for the last one
    (4, 9, 8, 4, 767),       # more workgroups, fewer ranges
])
def test_decode_attention_over_ranges_of_keys(T, b, heads, kv_heads, L):
    cfg = _cfg(T, b, heads, T * 64, L, 0.5, kv_heads)
    d = make_inputs(cfg, seed=37, weight_std=0.05 if cfg.h < 4096 else 0.02)
    got = run_decode(cfg, d)
    ref = oracle_decode(cfg, d)
    assert_close(got["H"], ref["H"], "H", tol=1e-2)     # q, k, v and H are each rounded to bf16 once: 4 x 2^-9 at most
    assert_close(bits_to_f64(got["Kc_bits"][:, :, :, L]), ref["k_new"], "k_new")
    assert_close(bits_to_f64(got["Vc_bits"][:, :, :, L]), ref["v_new"], "v_new")
    assert np.array_equal(got["Kc_bits"][:, :, :, :L], d["Kc"][:, :, :, :L])
    assert np.array_equal(got["Vc_bits"][:, :, :, :L], d["Vc"][:, :, :, :L])


@pytest.mark.parametrize("kv_heads,L", [(0, 37), (2, 1023)])
def test_decode_attention_infinite_values(kv_heads, L):
    """An infinite element of a cached value makes that output element infinite for the query heads that attend to it
    (every probability here is positive) and touches nothing else."""
    cfg = _cfg(2, 3, 8, 2 * 256, L, 0.5, kv_heads)
    d = make_inputs(cfg, seed=41, weight_std=0.05)
    shape = (cfg.T, cfg.batch, cfg.n_heads // cfg.T, 128)
    want = run_decode(cfg, d)["H"].reshape(shape)
    grp = cfg.n_heads // cfg.kv_heads
    for m, sq, hd, key, dim, bits in ((0, 0, 0, 3, 5, 0x7F80), (1, 2, 0, L - 1, 127, 0xFF80), (0, 1, 0, 20, 64, 0x7F80)):
        d["Vc"][m, sq, hd, key, dim] = bits
        want[m, sq, hd * grp:(hd + 1) * grp, dim] = np.inf if bits == 0x7F80 else -np.inf
    # the infinities spread over the rest of the layer, so only the heads' outputs are compared
    assert np.array_equal(run_decode(cfg, d)["H"].reshape(shape), want)


def test_decode_attention_probabilities_keep_fp32():
    """Per sequence: a key with probability weight w < 1 and value 1, and two keys of weight 1 whose values are minus the
    first two bf16 parts of w, so that the output is what is left of w below them, at most 2^-18."""
    L, n = 3, 8
    kappa = np.unique(I.bf16_bits_to_f32(I.f32_to_bf16_bits(np.linspace(-7.0, -0.1, 4001).astype(np.float32))))
    w = np.exp(kappa.astype(np.float64) / np.sqrt(128.0))
    rnd = lambda x: bits_to_f64(I.f32_to_bf16_bits(x.astype(np.float32)))
    hi = rnd(w)
    lo = rnd(w - hi)
    rest = w - hi - lo
    pick = np.argsort(-np.abs(rest))[:n]
    cfg = _cfg(1, n, 1, 64, L, 0.0)
    d = make_inputs(cfg, seed=43)
    d["R"][:] = 0x3F80                     # ones: their RMSNorm rounds to one
    d["gamma_attn"][:] = 0x3F80
    for name in ("Wqkv", "Kc", "Vc"):
        d[name][:] = 0
    d["Wqkv"][0, 63, 0] = 0x3F80           # q = 1 in dimension 63, whose angle at position 3 is 3.5e-4: cos rounds to 1
    for sq, c in enumerate(pick):
        d["Kc"][0, sq, 0, 0, 63] = I.f32_to_bf16_bits(kappa[c:c + 1])[0]
        d["Vc"][0, sq, 0, :3, 0] = I.f32_to_bf16_bits(np.array([1.0, -hi[c], -lo[c]], dtype=np.float32))
    got = run_decode(cfg, d)["H"][0, :, 0]
    want = rest[pick] / (3.0 + w[pick])    # the token's own key has weight 1 too and a value of zero
    # fp32: the score, its exponential and the sum are each off by at most about 2^-24; the output is rounded to bf16
    assert np.abs(got - want).max() <= 4 * 2.0 ** -24 / 3.0 + np.abs(want).max() * 2.0 ** -8
    assert np.abs(want).min() >= 2.0 ** -21


@pytest.mark.parametrize("scratch", ["whole", "two ranges of keys", "one range", "none"])
def test_decode_steps_on_one_workspace(scratch):
    """A workspace sized at the first step serves every length of the cache, through several numbers of key ranges, and
    smaller batches; one that ends anywhere in the scratch is good for the same results, with fewer ranges and the
    reduce + norm in place.  Nothing is written behind it."""
    import torch
    first = _cfg(4, 2, 12, 4 * 128, 0, 0.5)
    L = B.workspace_layout(B.make_desc(first))
    row = 4 * 2 * 3 * (128 + 4) * 4            # partial results of one range for all query heads
    spread = 4 * 2 * first.h * 2               # the o_proj output of the reduce + norm per (token, rank)
    assert row < spread < 2 * row < L.bytes_scratch
    size = {"whole": L.total_bytes, "two ranges of keys": L.off_scratch + 2 * row, "one range": L.off_scratch + row,
            "none": L.off_scratch}[scratch]
    guarded = torch.full((size + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    for batch, length in ((2, 0), (2, 15), (2, 140), (2, 700), (1, 700), (2, 1600), (2, 2500)):
        cfg = _cfg(4, batch, 12, 4 * 128, length, 0.5)
        d = make_inputs(cfg, seed=47, weight_std=0.05)
        got = run_decode(cfg, d, ws=guarded[:size])
        ref = oracle_decode(cfg, d)
        for name in ("X1", "H", "R1", "X2", "R2"):
            assert_close(got[name], ref[name], name)
        assert bool((guarded[size:] == 0xA5).all())
    with pytest.raises(B.CaatError) as e:
        run_decode(first, make_inputs(first, seed=47), ws=guarded[:L.off_scratch - 1])
    assert e.value.status == B.EWORKSPACE
