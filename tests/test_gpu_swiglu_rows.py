"""SwiGLU in the epilogue of the streaming gate/up GEMM (wide feed-forward blocks, up to 64 rows), whose waves finish 16 features each:
row counts at the edges of a 32-row and of a 64-row tile, two to four waves per workgroup.  Bounds: the layer parity tests'."""
import pytest

import workload as W
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("ffn", [8192, 10240, 16384])  # two, three and four waves
@pytest.mark.parametrize("tree,batches", [(W.TREE1, [1, 15, 16, 17, 31, 32, 33, 63, 64]), (W.TREE15, [1, 2, 3, 4]), (W.TREE64, [1])],
                         ids=["1 node", "15 nodes", "64 nodes"])
def test_layer_with_a_wide_feed_forward_block(tree, batches, ffn, dtype):
    w = W.CONFIGS["cfg2_layer_bf16"].with_(d=256, n_heads=2, head_dim=128, ffn=ffn, dtype=dtype, tree=tree, name=f"wide_ffn_{tree.name}")
    for n in batches:
        S_list = [(7 * b) % 40 for b in range(n)]
        _check_layer(_layer_case(w, S_list, 40, x_seed=f"wide_ffn_x{n}"), S_list, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("ffn", [5056, 5120, 8192, 8256, 10272, 11008, 12288, 12320, 16384, 32768])
def test_waves_per_workgroup(ffn, dtype):
    """5056: too few columns; 5120 .. 8192: two waves; 8256: three; 10272: an odd number of gate/up tile pairs, which the fused launch does not take; 11008: 688 waves of 32 columns, 229 workgroups of
    three and one with a single one; 12288: 768, the most that three waves serve; 12320 not fused; 16384, 32768: four waves, one band
    and two bands per workgroup."""
    w = W.CONFIGS["cfg2_layer_bf16"].with_(d=256, n_heads=2, head_dim=128, ffn=ffn, dtype=dtype, tree=W.TREE15, name=f"swiglu_waves_{ffn}")
    for n in (2, 3):
        S_list = [(7 * b) % 40 for b in range(n)]
        _check_layer(_layer_case(w, S_list, 40, x_seed=f"swiglu_waves_x{n}"), S_list, dtype)
