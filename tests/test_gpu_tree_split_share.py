"""Tree attention with one or two prefix splits, where the split of the tree slots also takes the end of the prefix: lengths around the
blocks of 32 keys at which its share begins (it takes its first block of 26 with one prefix split and of 51 with two; of 34 and 67 with
8-bit rows) and grows, with and without a tree slot in the shared block, beside short and empty prefixes in the same launch.
Batch x heads chooses the number of splits in a launch planned for 2048 keys or more.  Bounds: the layer parity tests'."""
import pytest

import workload as W
from tests import gpu_util as G
from tests.test_gpu_kv8 import check_layer_kv8
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu


def _case(batch, first, **kw):
    """first: whole prefix blocks that the lengths lie around."""
    w = W.CONFIGS["cfg2_layer_bf16"].with_(d=256, n_heads=2, head_dim=128, ffn=704, name=f"share_{first}", **kw)
    begin = 32 * first
    lengths = [0, 1, 31, begin - 64, begin - 1, begin, begin + 1, begin + 31, begin + 32, begin + 63, begin + 96, begin + 159, begin + 250]
    S_list = [lengths[(5 * b) % len(lengths)] if b % 3 == 0 else 7 * b for b in range(batch)]
    assert set(lengths) <= set(S_list)
    max_prefix = max(2100, max(S_list))
    assert G.attention_plan(w, batch, max_prefix)["splits"] == (2 if batch == 48 else 3)  # one of them the tree's
    return w, S_list, max_prefix


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("batch,first", [(48, 26), (40, 51), (48, 32), (40, 64)])
def test_layer_around_the_share(dtype, batch, first):
    w, S_list, max_prefix = _case(batch, first, dtype=dtype)
    _check_layer(_layer_case(w, S_list, max_prefix, x_seed=f"share_x{batch}"), S_list, dtype)


@pytest.mark.parametrize("batch,first", [(48, 34), (40, 67)])
def test_layer_around_the_share_8bit(batch, first):
    w, S_list, max_prefix = _case(batch, first, kv_quant="fp8e4m3")
    w = w.with_(prefix=tuple(S_list))
    check_layer_kv8(_layer_case(w, S_list, max_prefix, x_seed=f"share8_x{batch}"), S_list, w, f"share8_x{batch}")
