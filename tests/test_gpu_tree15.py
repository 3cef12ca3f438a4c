"""The 15-node tree at head_dim 128 in the 16-bit types: its attention runs the matrix-core kernel with 15 of 32 query rows in
use.  Prefix lengths around the key-block edges (the tree's slots then fall into one block or two), several key-splits, a
ragged batch with an empty prefix, grouped heads, and the order with a separate RoPE + cache-write kernel.
Bounds: those of the layer parity tests."""
import pytest

import paper_2603_03383_amd as P
import workload as W
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu


def _w(dtype="bf16", **kw):
    return W.CONFIGS["cfg2_layer_bf16"].with_(**{**dict(d=512, n_heads=4, head_dim=128, ffn=704, dtype=dtype, tree=W.TREE15,
                                                        name="tree15_layer"), **kw})


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("S_list,max_prefix", [([0], 0), ([1], 5), ([17], 17), ([18], 20), ([31], 31), ([32], 40),
                                               ([300, 0, 45], 300), ([5000, 131], 5003)], ids=str)
def test_layer(dtype, S_list, max_prefix):
    r = _layer_case(_w(dtype), S_list, max_prefix, x_seed=f"t15_{len(S_list)}")
    _check_layer(r, S_list, dtype)


def test_grouped_heads():
    r = _layer_case(_w("fp16", n_kv_heads=2, name="tree15_gqa"), [77, 640], 700, x_seed="t15_gqa")
    _check_layer(r, [77, 640], "fp16")


def test_separate_rope_kernel():
    was = P.medusa_test_force_unfused_rope(True)
    try:
        for S_list in ([0], [33], [300, 0, 45]):
            r = _layer_case(_w(), S_list, max(S_list), x_seed=f"t15u_{len(S_list)}")
            _check_layer(r, S_list, "bf16")
    finally:
        P.medusa_test_force_unfused_rope(was)
