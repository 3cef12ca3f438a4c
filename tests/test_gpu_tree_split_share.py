"""Tree attention with one or two prefix splits, where the split of the tree slots also takes the end of the prefix: lengths around the
blocks at which its share begins (32 and 64 blocks of 32 keys) and grows, with and without a tree slot in the shared block, beside
short and empty prefixes in the same launch.  Batch x heads chooses the number of splits.  Bounds: the layer parity tests'."""
import pytest

import workload as W
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("batch,edge", [(48, 32), (40, 64)])
def test_layer_around_the_share(dtype, batch, edge):
    w = W.CONFIGS["cfg2_layer_bf16"].with_(d=256, n_heads=2, head_dim=128, ffn=704, dtype=dtype, name=f"share_{edge}")
    lengths = [0, 1, 31, 32 * edge - 1, 32 * edge, 32 * edge + 1, 32 * edge + 63, 32 * edge + 64, 32 * edge + 96, 32 * edge + 159,
               32 * edge + 160, 32 * edge + 250]
    S_list = [lengths[(5 * b) % len(lengths)] if b % 4 == 0 else 7 * b for b in range(batch)]
    S_list[-1] = lengths[-1]
    _check_layer(_layer_case(w, S_list, max(S_list), x_seed=f"share_x{batch}"), S_list, dtype)
