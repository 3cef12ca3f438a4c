"""The tree's own K and V rows in the fused tree attention: they enter the product from LDS and reach the cache as whole 1 KiB units
that may also hold prefix keys or slots behind the tree.  Lengths that put the first and last tree slot on every kind of place in
a block of 32 keys; sequences beside each other; more partial-sum slots than are requested together (narrow models); grouped heads
(one workgroup of a group writes); both numbers of queries per workgroup.  Output, tree rows and the untouched prefix rows are
checked; bounds: the layer parity tests'."""
import pytest

import paper_2603_03383_amd as P
import workload as W
from tests.test_gpu_kv8 import check_layer_kv8
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 3, 4, 15, 17, 31, 32, 33, 49, 63, 97]


def _w(tree, dtype="bf16", n_heads=4, **kw):
    return W.CONFIGS["cfg2_layer_bf16"].with_(d=128 * n_heads, n_heads=n_heads, head_dim=128, ffn=704, dtype=dtype, tree=tree,
                                              name=f"rows_{tree.name}_{n_heads}", **kw)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("tree", [W.TREE15, W.TREE64], ids=lambda t: t.name)
@pytest.mark.parametrize("n_heads,kv_heads", [(4, 0), (8, 2)])
def test_layer_rows_at_block_edges(tree, dtype, n_heads, kv_heads):
    w = _w(tree, dtype, n_heads, n_kv_heads=kv_heads)
    for S in EDGES:
        _check_layer(_layer_case(w, [S], 97, x_seed=f"rows_x{S}"), [S], dtype)
    _check_layer(_layer_case(w, EDGES, 97, x_seed="rows_xb"), EDGES, dtype)


@pytest.mark.parametrize("max_prefix", [97, 14400], ids=["32 queries", "64 queries"])
def test_layer_rows_at_block_edges_8bit(max_prefix):
    w = _w(W.TREE64, n_kv_heads=2, kv_quant="fp8e4m3")
    for S in (0, 1, 15, 31, 33, 63):
        check_layer_kv8(_layer_case(w.with_(prefix=(S,)), [S], max_prefix, x_seed=f"rows8_x{S}"), [S], w.with_(prefix=(S,)), f"rows8_x{S}")


def test_layer_rows_with_64_queries_per_workgroup():
    w = _w(W.TREE64)
    for S in (0, 17, 33):
        _check_layer(_layer_case(w, [S], 4000, x_seed=f"rows64_x{S}"), [S], "bf16")


def test_the_narrow_models_have_more_slots_than_are_requested_together():
    assert P.medusa_gemm_plan(P.MDZ_BF16, 64, 3 * 512, 512, 12)["max_slots"] > 2
