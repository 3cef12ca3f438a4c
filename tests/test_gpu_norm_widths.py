"""Residual update + RMSNorm over widths around the vector kernel's edges: a part of one wave, no whole number of waves, the last
width of one float4 per thread and the first of two, its last width and the first one beyond it (the element-wise kernel).
Bounds: the layer parity tests'."""
import pytest

import workload as W
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu


WIDTHS = [("bf16", 1, 32), ("fp16", 9, 32), ("bf16", 65, 32), ("bf16", 16, 128), ("bf16", 129, 32), ("fp16", 40, 128), ("bf16", 64, 128),
          ("bf16", 257, 32), ("fp32", 1, 16), ("fp32", 4, 20), ("fp32", 258, 16)]


# (binary16 feed-forward operands are an option of bf16 models)
@pytest.mark.parametrize("dtype,n_heads,head_dim,ffn_f16", [(*w, f) for w in WIDTHS for f in (False, True) if not f or w[0] == "bf16"])
def test_layer(dtype, n_heads, head_dim, ffn_f16):
    ffn = 384 if dtype != "fp32" else 48
    w = W.CONFIGS["cfg2_layer_bf16"].with_(d=n_heads * head_dim, n_heads=n_heads, head_dim=head_dim, ffn=ffn, dtype=dtype, tree=W.TREE15,
                                           ffn_f16=ffn_f16, name=f"norm_{n_heads * head_dim}")
    _check_layer(_layer_case(w, [5, 40], 40, x_seed=f"norm_x{n_heads}"), [5, 40], dtype)
