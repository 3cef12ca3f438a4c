"""Key-splits and queries per workgroup of the tree attention (attn_plan in attn_mfma.hip) at the lengths where the plan changes: 32 queries
per workgroup up to 96 MB of K and V (5859 keys of 32 heads, 14772 in 8-bit rows), 64 beyond; up to twelve splits of few heads; the 15-node
tree.  Every case asserts the plan it is written for.  Bounds: the layer parity tests'."""
import pytest

import workload as W
from tests import gpu_util as G
from tests.test_gpu_kv8 import check_layer_kv8
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu


def _w(n_heads, dtype="bf16", tree=W.TREE64, **kw):
    return W.CONFIGS["cfg2_layer_bf16"].with_(d=128 * n_heads, n_heads=n_heads, head_dim=128, ffn=704, dtype=dtype, tree=tree,
                                              name=f"plan_{tree.name}_{n_heads}", **kw)


def _plan(w, batch, max_prefix):
    p = G.attention_plan(w, batch, max_prefix)
    return p["queries"], p["splits"]


@pytest.mark.parametrize("n_heads,kv_heads,max_prefix,plan", [
    (32, 0, 5859, (32, 4)), (32, 0, 5860, (64, 6)), (16, 0, 11718, (32, 7)), (16, 0, 11719, (64, 10)), (16, 0, 16384, (64, 12)), (40, 0, 4000, (32, 3)),
    (32, 8, 11718, (32, 4)), (32, 8, 11719, (64, 8)), (4, 0, 4000, (32, 4))])
def test_one_sequence(n_heads, kv_heads, max_prefix, plan):
    w = _w(n_heads, n_kv_heads=kv_heads)
    assert _plan(w, 1, max_prefix) == plan
    for S in (max_prefix, 33):
        _check_layer(_layer_case(w, [S], max_prefix, x_seed=f"plan_x{n_heads}_{max_prefix}_{S}"), [S], "bf16")


@pytest.mark.parametrize("kv_heads,max_prefix,plan", [(0, 9000, (32, 4)), (0, 14773, (64, 8)), (8, 12543, (32, 4)), (8, 12544, (32, 8))])
def test_one_sequence_8bit(kv_heads, max_prefix, plan):
    S = 2000
    w = _w(32, kv_quant="fp8e4m3", n_kv_heads=kv_heads).with_(prefix=(S,))
    assert _plan(w, 1, max_prefix) == plan
    check_layer_kv8(_layer_case(w, [S], max_prefix, x_seed=f"plan8_x{max_prefix}"), [S], w, f"plan8_x{max_prefix}")


@pytest.mark.parametrize("n_heads,batch,max_prefix,splits", [(2, 3, 22000, 10), (32, 3, 9000, 2), (32, 5, 5000, 1)])
def test_several_sequences_8bit(n_heads, batch, max_prefix, splits):
    """32 queries per workgroup whatever the length."""
    S_list = [1300, 0, 700, 33, 64][:batch]
    w = _w(n_heads, kv_quant="fp8e4m3").with_(prefix=tuple(S_list))
    assert _plan(w, batch, max_prefix) == (32, splits)
    seed = f"plan8_x{n_heads}_{batch}"
    check_layer_kv8(_layer_case(w, S_list, max_prefix, x_seed=seed), S_list, w, seed)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("n_heads,batch,lengths,splits", [
    (32, 1, [1200], 6), (32, 3, [1184, 32, 700], 4), (32, 4, [200, 1000, 0, 31], 2), (2, 48, None, 4), (2, 49, None, 2), (2, 2, [4100, 40], 6),
    (16, 5, [2560, 100, 0, 31, 700], 3), (16, 3, [2561, 64, 33], 5), (2, 1, [16384], 9)])
def test_15_nodes(n_heads, batch, lengths, splits, dtype):
    w = _w(n_heads, dtype, W.TREE15)
    S_list = lengths or [(131 * b) % 1200 for b in range(batch)]
    assert _plan(w, batch, max(S_list)) == (32, splits)
    _check_layer(_layer_case(w, S_list, max(S_list), x_seed=f"plan15_x{batch}"), S_list, dtype)
