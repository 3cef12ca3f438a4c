"""Batches whose attention starts the longest sequences first (more workgroups than run at once and a long prefix bound): the
single-query kernels with grouped and ungrouped heads, the 15-node tree, the 64-node tree split and unsplit, with 8-bit rows; equal
lengths among them, and more than one group of 64 sequences.  Bounds: those of the layer parity tests."""
import numpy as np
import pytest

import workload as W
from tests import gpu_util as G
from tests.test_gpu_ar_attention import EDGES
from tests.test_gpu_kv8 import KV8_DIRECT_TOL
from tests.test_gpu_parity import _check_layer, _layer_case, _scale

pytestmark = pytest.mark.gpu


def _w(tree, n_heads, kv_heads, dtype="bf16", **kw):
    return W.CONFIGS["cfg2_layer_bf16"].with_(d=128 * n_heads, n_heads=n_heads, n_kv_heads=kv_heads, head_dim=128, ffn=704, dtype=dtype,
                                              tree=tree, name=f"order_{tree.name}_{n_heads}_{kv_heads}", **kw)


def _run(w, S_list, max_prefix, splits, kernel="tree", queries=32):
    assert G.attention_plan(w, len(S_list), max_prefix) == dict(kernel=kernel, queries=queries, splits=splits, ordered=True)
    r = _layer_case(w, S_list, max_prefix, x_seed=f"order_x{len(S_list)}")
    if w.kv_quant:  # (codes may land on the neighbouring value)
        assert np.abs(r["x"] - r["ref"]).max() <= KV8_DIRECT_TOL[w.dtype] * _scale(r["ref"])
    else:
        _check_layer(r, S_list, w.dtype)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("n_heads,kv_heads,splits,kernel", [(16, 8, 4, "one_mfma"), (32, 32, 3, "one_fma")])  # x 136 and 544 workgroups
def test_single_query(dtype, n_heads, kv_heads, splits, kernel):
    _run(_w(W.TREE1, n_heads, kv_heads, dtype), EDGES[:-1] + [2310], 2310, splits, kernel, 1)


def test_fifteen_nodes_over_more_than_64_sequences():
    lengths = [7, 7, 1040, 31, 300, 0, 64]
    _run(_w(W.TREE15, 4, 4), [lengths[(3 * b) % 7] for b in range(70)], 1040, 1)


@pytest.mark.parametrize("quant", ["", "fp8e4m3"])
def test_sixty_four_nodes_unsplit(quant):
    lengths = [5, 90, 2600 if not quant else 1100, 90, 33]
    _run(_w(W.TREE64, 4, 4, kv_quant=quant), [lengths[(2 * b) % 5] if b % 16 == 0 else 3 * b for b in range(66)], max(lengths), 1,
         queries=64)


def test_sixty_four_nodes_split():
    _run(_w(W.TREE64, 32, 8, "fp16"), [200, 2100, 31], 2100, 2)
