"""Key-splits and kernel of the single-query attention (decode_splits in attn_decode.hip) at the lengths and batches where they change: one split
up to twelve blocks; several sequences of ungrouped heads, in the FMA kernel from seven blocks per split on; more pairs than CUs; grouped heads, a
workgroup per CU and two; 8-bit rows; K and V loaded non-temporally once a pass reads 350 MB of them.  Every case asserts the plan it is
written for.  Bounds: the layer parity tests'."""
import pytest

import workload as W
from tests import gpu_util as G
from tests.test_gpu_kv8 import check_layer_kv8
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu


def _w(n_heads, dtype="bf16", **kw):
    return W.CONFIGS["cfg2_layer_bf16"].with_(d=128 * n_heads, n_heads=n_heads, head_dim=128, ffn=704, dtype=dtype, tree=W.TREE1,
                                              name=f"decode_plan_{n_heads}", **kw)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("n_heads,kv_heads,batch,max_prefix,kernel,splits", [
    (4, 0, 1, 383, "one_mfma", 1), (4, 0, 1, 384, "one_mfma", 2),      # twelve blocks, thirteen
    (4, 0, 3, 3000, "one_mfma", 6),                                    # by length
    (2, 0, 48, 1119, "one_mfma", 3), (2, 0, 48, 1120, "one_fma", 6), (2, 0, 48, 2272, "one_fma", 6),
    (2, 0, 64, 895, "one_mfma", 2), (2, 0, 64, 896, "one_fma", 5),
    (2, 0, 112, 639, "one_mfma", 1), (2, 0, 112, 640, "one_fma", 3),   # nearly as many pairs as CUs
    (2, 0, 129, 2047, "one_fma", 2), (2, 0, 129, 2048, "one_fma", 3),  # more
    (2, 0, 260, 2048, "one_fma", 3),
    (4, 2, 64, 4095, "one_mfma", 2), (4, 2, 64, 4096, "one_mfma", 4),
    (4, 2, 68, 2303, "one_mfma", 1), (4, 2, 68, 2304, "one_mfma", 4),
    (4, 2, 129, 2047, "one_mfma", 1), (4, 2, 129, 2048, "one_mfma", 2),
    (4, 2, 8, 2064, "one_mfma", 8), (4, 2, 8, 3000, "one_mfma", 8),    # few pairs
])
def test_layer(n_heads, kv_heads, batch, max_prefix, kernel, splits, dtype):
    w = _w(n_heads, dtype, n_kv_heads=kv_heads)
    plan = G.attention_plan(w, batch, max_prefix)
    assert (plan["kernel"], plan["splits"]) == (kernel, splits)
    S_list = [max_prefix if batch == 1 else (611 * b) % min(1500, max_prefix) for b in range(batch)]
    S_list[-1] = min(max_prefix, 2000)
    _check_layer(_layer_case(w, S_list, max_prefix, x_seed=f"decode_plan_x{batch}_{max_prefix}"), S_list, dtype)


@pytest.mark.parametrize("kv_heads", [0, 8])
def test_non_temporal_loads(kv_heads):
    w = _w(32, n_kv_heads=kv_heads)
    max_prefix = 21400 if kv_heads == 0 else 85500
    for S in (31, 700):
        _check_layer(_layer_case(w, [S], max_prefix, x_seed=f"decode_nt_x{S}"), [S], "bf16")


def test_non_temporal_loads_8bit():
    w = _w(32, kv_quant="fp8e4m3").with_(prefix=(700,))
    check_layer_kv8(_layer_case(w, [700], 41500, x_seed="decode_nt8_x"), [700], w, "decode_nt8_x")


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("n_heads,kv_heads,batch,max_prefix,kernel,splits", [
    (2, 0, 48, 1119, "one_mfma", 3), (2, 0, 48, 1120, "one_fma", 6), (2, 0, 16, 3600, "one_fma", 17), (2, 0, 128, 640, "one_fma", 3),
    (4, 0, 1, 1400, "one_mfma", 6), (40, 0, 1, 3584, "one_fma", 13), (4, 2, 68, 2304, "one_mfma", 4), (4, 2, 48, 3584, "one_mfma", 6)])
def test_8bit_splits(n_heads, kv_heads, batch, max_prefix, kernel, splits, dtype):
    """Several sequences around the length where the FMA kernel takes them, in seventeen splits and at the most pairs; one sequence, a long one of
    40 heads; grouped heads from the lengths on where they take two workgroups per CU."""
    S_list = [(211 * b) % 600 for b in range(batch)]
    S_list[-1] = min(max_prefix, 1100)
    w = _w(n_heads, dtype, kv_quant="fp8e4m3", n_kv_heads=kv_heads).with_(prefix=tuple(S_list))
    seed = f"decode_plan8_x{batch}_{max_prefix}"
    plan = G.attention_plan(w, batch, max_prefix)
    assert (plan["kernel"], plan["splits"]) == (kernel, splits)
    check_layer_kv8(_layer_case(w, S_list, max_prefix, x_seed=seed), S_list, w, seed)
