"""Key-splits of the single-query attention (decode_splits in attn_decode.hip) at the lengths and batches where they change: one split up to
twelve blocks; many sequences of ungrouped heads, in the other kernel from 2048 keys on; grouped heads below and from 4096 keys on; K and V loaded
non-temporally once a pass reads 350 MB of them.  Bounds: the layer parity tests'."""
import pytest

import paper_2603_03383_amd as P
import workload as W
from tests.test_gpu_kv8 import check_layer_kv8
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu


def _w(n_heads, dtype="bf16", **kw):
    return W.CONFIGS["cfg2_layer_bf16"].with_(d=128 * n_heads, n_heads=n_heads, head_dim=128, ffn=704, dtype=dtype, tree=W.TREE1,
                                              name=f"decode_plan_{n_heads}", **kw)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("n_heads,kv_heads,batch,max_prefix", [
    (4, 0, 1, 383), (4, 0, 1, 384),        # twelve blocks, thirteen
    (4, 0, 3, 3000),                       # splits by length
    (2, 0, 48, 1119), (2, 0, 48, 1120),    # three splits; six, FMA kernel
    (2, 0, 64, 895), (2, 0, 64, 896),      # two; five, FMA kernel
    (2, 0, 112, 639), (2, 0, 112, 640),    # one; three, FMA kernel
    (2, 0, 129, 2047), (2, 0, 129, 2048),  # more pairs than CUs: two and three splits
    (2, 0, 260, 2048),                     # 520 pairs: three
    (4, 2, 64, 4095), (4, 2, 64, 4096),    # grouped: two and four splits
    (4, 2, 68, 2303), (4, 2, 68, 2304),    # one and four
    (4, 2, 129, 2047), (4, 2, 129, 2048),  # one and two
])
def test_layer(n_heads, kv_heads, batch, max_prefix, dtype):
    w = _w(n_heads, dtype, n_kv_heads=kv_heads)
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
@pytest.mark.parametrize("n_heads,kv_heads,batch,max_prefix,splits", [
    (2, 0, 48, 1119, 3), (2, 0, 48, 1120, 6), (2, 0, 16, 3600, 17), (2, 0, 128, 640, 3), (4, 0, 1, 1400, 6), (4, 2, 68, 2304, 4), (4, 2, 48, 3584, 6)])
def test_8bit_splits(n_heads, kv_heads, batch, max_prefix, splits, dtype):
    """Several sequences around the length where the FMA kernel takes them, in seventeen splits and at the most pairs; one sequence; grouped
    heads from the lengths on where they take two workgroups per CU."""
    S_list = [(211 * b) % 600 for b in range(batch)]
    S_list[-1] = min(max_prefix, 1100)
    w = _w(n_heads, dtype, kv_quant="fp8e4m3", n_kv_heads=kv_heads).with_(prefix=tuple(S_list))
    seed = f"decode_plan8_x{batch}_{max_prefix}"
    r = _layer_case(w, S_list, max_prefix, x_seed=seed)
    plan = P.medusa_attention_plan(r["kv"].model.desc, batch, max_prefix, "fp8e4m3")
    assert plan["splits"] == splits and plan["kernel"] == ("one_fma" if not kv_heads and splits * batch * n_heads > 512 else "one_mfma")
    check_layer_kv8(r, S_list, w, seed)
