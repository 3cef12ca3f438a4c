"""The single-query attention of ungrouped heads with more (sequence, head, split) workgroups than two per CU, which have a kernel of
their own: slot S at the places of its 32-key block that the own-row insertion tells apart, one and two key-splits, both 16-bit
types, 8-bit rows, the order with a separate RoPE kernel, a launch in length order and one of equal lengths.  Bounds: those of the
other single-query tests."""
import numpy as np
import pytest

import paper_2603_03383_amd as P
from tests.test_gpu_ar_attention import EDGES, _w
from tests.test_gpu_attention_precision import _check
from tests.test_gpu_parity import _check_layer, _layer_case, _scale

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("n_heads", [16, 32])  # 17 sequences: 2 x 272 and 544 workgroups
def test_slot_positions(dtype, n_heads):
    r = _layer_case(_w(dtype, n_heads, n_heads), EDGES, 1000, x_seed="pairs_edges")
    _check_layer(r, EDGES, dtype)


def test_equal_lengths_and_one_block():
    r = _layer_case(_w("bf16", 16, 16), [7] * 36, 7, x_seed="pairs_equal")
    _check_layer(r, [7] * 36, "bf16")


def test_separate_rope_kernel():
    was = P.medusa_test_force_unfused_rope(True)
    try:
        r = _layer_case(_w("fp16", 32, 32), EDGES, 1000, x_seed="pairs_unfused")
        _check_layer(r, EDGES, "fp16")
    finally:
        P.medusa_test_force_unfused_rope(was)


@pytest.mark.parametrize("n_heads", [16, 32])
def test_eight_bit_rows(n_heads):
    r = _layer_case(_w("fp16", n_heads, n_heads, kv_quant="fp8e4m3"), EDGES, 1000, x_seed="pairs_q8")
    # an 8-bit code may land on its neighbour (a grid step of 2^-3.5 with probability u / step): 2 sqrt(u 2^-3.5), u = 2^-12
    assert np.abs(r["x"] - r["ref"]).max() <= 9.3e-3 * _scale(r["ref"])


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("quant,v_std", [("", 1.0), ("fp8e4m3", 1.0), ("fp8e4m3", 1e-4)])
def test_softmax_weights_are_fp32(dtype, quant, v_std):
    _check("tree1", dtype, 8, 8, [(37 * b) % 300 for b in range(60)] + [40, 0, 5, 100, 640], 640, quant=quant, v_std=v_std)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("n_heads,lengths", [(8, EDGES), (9, EDGES[:15] * 4)], ids=["8x17", "9x60"])  # 540 workgroups: the FMA kernel
def test_more_partial_sums_than_are_requested_together(dtype, n_heads, lengths):
    """Narrow models: the QKV product comes in eight and nine slots, the kernels request four before the first K / V block."""
    d = 128 * n_heads
    assert P.medusa_gemm_plan(P.DTYPES[dtype], len(lengths), 3 * d, d, 12)["max_slots"] >= 8
    r = _layer_case(_w(dtype, n_heads, n_heads), lengths, 1000, x_seed="pairs_slots")
    _check_layer(r, lengths, dtype)
