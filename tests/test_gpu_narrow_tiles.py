"""Tiles of 96 columns (gemm_tile.hip: one block of up to 96 or 192 rows on at least 7/8 of the CUs): the gate/up product with its
mixed gate and up columns (22016 and 21504 columns, i.e. 229 1/3 and 224 column blocks) and a product split in two over K (128 blocks), at row
counts around the tiles' edges.  Every case asserts the tile it is written for.  Bounds: the layer parity tests'."""
import pytest

import paper_2603_03383_amd as P
import workload as W
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu


def _plan(w, rows, N, K, max_split, swiglu=False):
    p = P.medusa_gemm_many_rows_plan(P.DTYPES[w.dtype], rows, N, K, max_split, swiglu)
    return p["tile_rows"], p["tile_cols"], p["k_splits"]


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("d,ffn", [(256, 11008), (320, 10752)])
@pytest.mark.parametrize("tree,batch,tile_rows", [(W.TREE1, 65, 96), (W.TREE15, 6, 96), (W.TREE1, 96, 96), (W.TREE1, 129, 192), (W.TREE64, 3, 192)],
                         ids=lambda v: getattr(v, "name", v))
def test_gate_up(dtype, d, ffn, tree, batch, tile_rows):
    """Contractions of 4 and of 5 rounds (an even and an odd number, in a ring of four)."""
    w = W.CONFIGS["cfg2_layer_bf16"].with_(d=d, n_heads=d // 64, head_dim=64, ffn=ffn, dtype=dtype, tree=tree, name=f"narrow_tiles_{ffn}")
    assert _plan(w, batch * P.medusa_tree_info(P.TREES[tree.name])["T"], 2 * ffn, d, 1, True) == (tile_rows, 96, 1)
    S_list = [(5 * b + 2) % 30 for b in range(batch)]
    _check_layer(_layer_case(w, S_list, 30, x_seed=f"narrow_tiles_x{batch}"), S_list, dtype)


@pytest.mark.parametrize("tree,batch,tile_rows", [(W.TREE15, 5, 96), (W.TREE15, 12, 192)], ids=lambda v: getattr(v, "name", v))
def test_split_product(tree, batch, tile_rows):
    w = W.CONFIGS["cfg2_layer_bf16"].with_(ffn=512, tree=tree, name="narrow_tiles_qkv")
    assert _plan(w, batch * 15, 3 * w.d, w.d, 12) == (tile_rows, 96, 2)
    S_list = [(5 * b + 2) % 30 for b in range(batch)]
    _check_layer(_layer_case(w, S_list, 30, x_seed=f"narrow_tiles_qkv_x{batch}"), S_list, "bf16")
