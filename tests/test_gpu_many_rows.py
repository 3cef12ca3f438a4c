"""Layers over more than 64 rows (several sequences, gemm_tile.hip): row counts around the edges of the row tiles and blocks
(65 .. 513), matrices whose last column block is ragged, contractions of a few rounds only, every tree, both 16-bit types.
Bounds: those of the layer parity tests (bf16 2e-2 of the output scale, fp16 2e-2 x 2^-3)."""
import pytest

import workload as W
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("tree,batch", [(W.TREE1, 65), (W.TREE15, 5), (W.TREE15, 6), (W.TREE1, 97), (W.TREE1, 127),
                                        (W.TREE64, 2), (W.TREE15, 9), (W.TREE64, 3), (W.TREE1, 193), (W.TREE1, 257),
                                        (W.TREE64, 5), (W.TREE64K5, 8), (W.TREE1, 513)],
                         ids=lambda v: getattr(v, "name", v))
def test_layer_over_many_rows(dtype, tree, batch):
    w = W.CONFIGS["cfg2_layer_bf16"].with_(d=256, n_heads=2, head_dim=128, ffn=704, dtype=dtype, tree=tree,
                                           name=f"rows_{tree.name}_{batch}")
    S_list = [(37 * b + 5) % 90 for b in range(batch)]
    r = _layer_case(w, S_list, 90, x_seed=f"rows_x{batch}")
    _check_layer(r, S_list, dtype)


@pytest.mark.parametrize("d,n_heads,head_dim,ffn", [(320, 5, 64, 352), (64, 1, 64, 64), (1152, 9, 128, 1088)])
def test_ragged_column_blocks_and_short_contractions(d, n_heads, head_dim, ffn):
    """QKV widths of 7.5, 1.5 and 27 column blocks of 128, contractions of 5, 1 and 18 rounds; ffn 352 is no whole number of
    rounds, so its down projection takes the portable kernel."""
    w = W.CONFIGS["cfg2_layer_bf16"].with_(d=d, n_heads=n_heads, head_dim=head_dim, ffn=ffn, tree=W.TREE15, name=f"ragged_{d}")
    S_list = [0, 3, 40, 17, 64, 33]
    r = _layer_case(w, S_list, 64, x_seed=f"ragged_x{d}")
    _check_layer(r, S_list, "bf16")
