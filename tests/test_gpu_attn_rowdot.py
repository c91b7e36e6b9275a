"""The sums dO * O of the attention backward, made by the dQ kernel for the dK / dV kernel or, up to 256 workgroups of dK / dV, in
front of both in one launch: sequences that end inside a block of queries on a workspace full of NaN give the bits they give on a
cleared one, and the oracle's gradients."""
import numpy as np
import pytest

from tests.test_gpu_attn import _cfg, check_attn_bwd, oracle_attn_block, oracle_attn_bwd, run_attn_block
from tests.util import make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,heads,kv,batch,seq", [(2, 4, 4, 1, 1), (2, 4, 2, 3, 63), (1, 4, 1, 2, 65), (2, 4, 4, 1, 128), (2, 8, 4, 2, 129),
                                                  (1, 8, 1, 1, 190), (4, 8, 8, 1, 257),
                                                  (2, 4, 4, 64, 127), (2, 4, 4, 65, 100), (2, 4, 4, 35, 191), (1, 8, 2, 129, 65),
                                                  (1, 4, 1, 260, 1), (2, 8, 4, 22, 257)])
def test_row_sums_on_a_workspace_of_nan(T, heads, kv, batch, seq, monkeypatch):
    import torch
    cfg = _cfg(T, batch, seq, heads, 0.5, kv_heads=kv)
    d = make_inputs(cfg, seed=51, with_grads=True, weight_std=0.05)
    clear = run_attn_block(cfg, d, backward=True)
    monkeypatch.setattr(torch, "zeros", lambda n, **kw: torch.full((n,), 255, **kw))     # the helper's workspace
    got = run_attn_block(cfg, d, backward=True)
    for name in ("dqkv", "dX", "dR", "dWqkv", "dWo"):
        assert np.array_equal(got[name], clear[name]), name
    w, fwd = oracle_attn_block(cfg, d)
    check_attn_bwd(got, oracle_attn_bwd(cfg, w, fwd))
