"""Short sequences in a launch planned for a long prefix: the key-splits of the tree attention are chosen by max_prefix, so most of
them get no block of a short sequence, and the merge, which takes the splits eight at a time, meets a whole group of empty ones
before the split of the tree slots (9 to 12 splits at 16384 keys, 10 to 12 at 20736).  Both 16-bit types and both orders of RoPE; lengths
around the first two key blocks.  Bounds: the layer parity tests'."""
import pytest

import paper_2603_03383_amd as P
import workload as W
from tests import gpu_util as G
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu

SHORT = [0, 20, 31, 40, 63]


def _w(tree, n_heads, dtype="bf16", **kw):
    return W.CONFIGS["cfg2_layer_bf16"].with_(d=128 * n_heads, n_heads=n_heads, head_dim=128, ffn=704, dtype=dtype, tree=tree,
                                              name=f"short_{tree.name}_{n_heads}", **kw)


def _run(w, S_list, max_prefix, fused=True):
    assert G.attention_plan(w, len(S_list), max_prefix, fused)["splits"] >= 9
    r = _layer_case(w, S_list, max_prefix, x_seed=f"short_x{max_prefix}_{len(S_list)}")
    _check_layer(r, S_list, w.dtype)


# (one sequence at a time: 64 rows at most)
@pytest.mark.parametrize("S", SHORT)
@pytest.mark.parametrize("max_prefix", [16384, 20736])
@pytest.mark.parametrize("n_heads", [2, 16])
@pytest.mark.parametrize("tree", [W.TREE15, W.TREE64], ids=lambda t: t.name)
def test_layer(tree, n_heads, max_prefix, S):
    _run(_w(tree, n_heads), [S], max_prefix)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
def test_ragged_batch(dtype):
    _run(_w(W.TREE15, 2, dtype), [40, 0, 700, 63], 20736)


@pytest.mark.parametrize("tree", [W.TREE15, W.TREE64], ids=lambda t: t.name)
def test_separate_rope_kernel(tree):
    was = P.medusa_test_force_unfused_rope(True)
    try:
        for S in (0, 40):
            _run(_w(tree, 2), [S], 20736, fused=False)
    finally:
        P.medusa_test_force_unfused_rope(was)
