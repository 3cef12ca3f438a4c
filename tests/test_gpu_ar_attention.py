"""The single-query attention where it can go wrong: slot S at every place of its 32-key block that the kernel's own-row
insertion tells apart (both half-waves, both halves of the block, first and last key), one to many key-splits, groups of 1 to
40 query heads (more than one column block), both 16-bit types, 8-bit rows, and the order with a separate RoPE kernel.
Bounds: those of the layer parity tests; 8-bit rows: the direct bound of their own tests."""
import pytest

import paper_2603_03383_amd as P
import workload as W
from tests.test_gpu_parity import TOL, _check_layer, _layer_case, _scale

import numpy as np

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 3, 4, 7, 8, 12, 15, 16, 20, 27, 31, 32, 63, 64, 230, 1000]


def _w(dtype, n_heads, kv_heads, **kw):
    return W.CONFIGS["cfg2_layer_bf16"].with_(d=128 * n_heads, n_heads=n_heads, n_kv_heads=kv_heads, head_dim=128, ffn=704,
                                              dtype=dtype, tree=W.TREE1, name=f"ar_{n_heads}_{kv_heads}", **kw)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("n_heads,kv_heads", [(2, 2), (4, 1), (16, 2), (40, 1)])
def test_slot_positions_and_groups(dtype, n_heads, kv_heads):
    r = _layer_case(_w(dtype, n_heads, kv_heads), EDGES, 1000, x_seed="ar_edges")
    _check_layer(r, EDGES, dtype)


@pytest.mark.parametrize("S,max_prefix", [(6000, 6000), (500, 6000), (0, 6000)])
def test_many_splits(S, max_prefix):
    r = _layer_case(_w("bf16", 2, 1), [S], max_prefix, x_seed="ar_splits")
    _check_layer(r, [S], "bf16")


def test_separate_rope_kernel():
    was = P.medusa_test_force_unfused_rope(True)
    try:
        r = _layer_case(_w("fp16", 8, 2), EDGES, 1000, x_seed="ar_unfused")
        _check_layer(r, EDGES, "fp16")
    finally:
        P.medusa_test_force_unfused_rope(was)


def test_eight_bit_rows():
    r = _layer_case(_w("fp16", 8, 2, kv_quant="fp8e4m3"), EDGES, 1000, x_seed="ar_q8")
    # an 8-bit code may land on its neighbour (a grid step of 2^-3.5 with probability u / step): 2 sqrt(u 2^-3.5), u = 2^-12
    assert np.abs(r["x"] - r["ref"]).max() <= 9.3e-3 * _scale(r["ref"])
