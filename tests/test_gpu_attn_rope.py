"""The rotary embedding at other bases, in the attention block's projections and, transposed, in its gradients: sequences that end
inside a tile of queries, of keys and of the GEMM's rows, one, several and 16 query heads per key head."""
import pytest

from tests.test_gpu_attn import _cfg, check_attn, check_attn_bwd, oracle_attn_block, oracle_attn_bwd, run_attn_block
from tests.util import make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,heads,kv,batch,seq,base", [
    (2, 4, 4, 1, 1, 1e4), (2, 4, 2, 3, 33, 1.5), (1, 4, 1, 2, 129, 5e5), (2, 8, 4, 3, 200, 0.5), (1, 16, 1, 1, 321, 1e4),
    (4, 8, 4, 1, 700, 1e2), (2, 2, 2, 1, 1025, 1e4)])
def test_attention_block_rotation(T, heads, kv, batch, seq, base):
    cfg = _cfg(T, batch, seq, heads, 0.5, kv_heads=kv).with_(rope_base=base)
    d = make_inputs(cfg, seed=41, with_grads=True, weight_std=0.05)
    got = run_attn_block(cfg, d, backward=True)
    w, fwd = oracle_attn_block(cfg, d)
    check_attn(cfg, d, got, fwd)
    check_attn_bwd(got, oracle_attn_bwd(cfg, w, fwd))
