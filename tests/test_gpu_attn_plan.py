"""Key-splits and queries per workgroup of the tree attention (attn_plan in attn_mfma.hip) at the lengths where the plan changes: 32 queries
per workgroup up to 96 MB of K and V (5859 keys of 32 heads, 14772 in 8-bit rows), 64 beyond; up to twelve splits of few heads; six splits
of the 15-node tree; several sequences in a launch planned for a longer prefix, whose tree split takes a share of the prefix.  Bounds: the layer
parity tests'."""
import pytest

import workload as W
from tests.test_gpu_kv8 import check_layer_kv8
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu


def _w(n_heads, dtype="bf16", tree=W.TREE64, **kw):
    return W.CONFIGS["cfg2_layer_bf16"].with_(d=128 * n_heads, n_heads=n_heads, head_dim=128, ffn=704, dtype=dtype, tree=tree,
                                              name=f"plan_{tree.name}_{n_heads}", **kw)


@pytest.mark.parametrize("n_heads,kv_heads,max_prefix", [
    (32, 0, 5859),    # 32 queries per workgroup, four splits
    (32, 0, 5860),    # 64 queries, six
    (16, 0, 11718),   # 32 queries, eight
    (16, 0, 11719),   # 64 queries, ten
    (40, 0, 4000),    # 32 queries, three
    (32, 8, 14648),   # grouped heads: 32 queries, four
    (32, 8, 14649),   # 64 queries, eight
    (4, 0, 4000),     # 32 queries, four by length
])
def test_one_sequence(n_heads, kv_heads, max_prefix):
    w = _w(n_heads, n_kv_heads=kv_heads)
    for S in (max_prefix, 33):
        _check_layer(_layer_case(w, [S], max_prefix, x_seed=f"plan_x{n_heads}_{max_prefix}_{S}"), [S], "bf16")


@pytest.mark.parametrize("max_prefix", [9000, 16384])
def test_one_sequence_8bit(max_prefix):
    S = 2000
    w = _w(32, kv_quant="fp8e4m3").with_(prefix=(S,))
    check_layer_kv8(_layer_case(w, [S], max_prefix, x_seed=f"plan8_x{max_prefix}"), [S], w, f"plan8_x{max_prefix}")


@pytest.mark.parametrize("n_heads,batch,max_prefix", [(2, 3, 22000), (32, 3, 9000), (32, 5, 5000)])
def test_several_sequences_8bit(n_heads, batch, max_prefix):
    """32 queries per workgroup whatever the length; ten splits, two and one."""
    S_list = [1300, 0, 700, 33, 64][:batch]
    w = _w(n_heads, kv_quant="fp8e4m3").with_(prefix=tuple(S_list))
    seed = f"plan8_x{n_heads}_{batch}"
    check_layer_kv8(_layer_case(w, S_list, max_prefix, x_seed=seed), S_list, w, seed)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("n_heads,batch,lengths", [(32, 1, [1200]), (32, 3, [1184, 32, 700]), (32, 4, [200, 1000, 0, 31]), (2, 48, None), (2, 49, None),
                                                   (2, 2, [4100, 40]), (16, 5, [2560, 100, 0, 31, 700]), (16, 3, [2561, 64, 33])])
def test_15_nodes(n_heads, batch, lengths, dtype):
    w = _w(n_heads, dtype, W.TREE15)
    S_list = lengths or [(131 * b) % 1200 for b in range(batch)]
    _check_layer(_layer_case(w, S_list, max(S_list), x_seed=f"plan15_x{batch}"), S_list, dtype)


def _share(batch, first, **kw):
    """Lengths around whole prefix block `first`, from where on the tree's split takes a share of the prefix."""
    w = _w(2, **kw)
    begin = 32 * first
    lengths = [0, 1, 31, begin - 64, begin - 1, begin, begin + 1, begin + 31, begin + 32, begin + 63, begin + 96, begin + 159, begin + 250]
    return w, [lengths[(5 * b) % len(lengths)] if b % 3 == 0 else 7 * b for b in range(batch)]


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("batch,first", [(48, 26), (40, 51), (48, 32)])  # two and three splits from 2048 keys on
def test_share_of_the_tree_split(batch, first, dtype):
    w, S_list = _share(batch, first, dtype=dtype)
    _check_layer(_layer_case(w, S_list, 2100, x_seed=f"plan_share_x{batch}"), S_list, dtype)


def test_share_of_the_tree_split_8bit():
    w, S_list = _share(48, 34, kv_quant="fp8e4m3")
    w = w.with_(prefix=tuple(S_list))
    check_layer_kv8(_layer_case(w, S_list, 2100, x_seed="plan_share8_x"), S_list, w, "plan_share8_x")
