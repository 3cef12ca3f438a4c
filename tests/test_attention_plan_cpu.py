"""CPU tests of the attention's host-side plan (no GPU work; 256 CUs): kernel, queries per workgroup, key-splits and the order of the
sequences."""
import pytest

import paper_2603_03383_amd as P


def _model(n_heads, kv_heads=0, tree="tree64", head_dim=128, dtype="bf16"):
    return P.ModelDesc(n_heads * head_dim, n_heads, head_dim, 704, 1024, 2, P.DTYPES[dtype], P.TREES[tree], 1e-5, 1e4, kv_heads)


def _plan(m, B, max_prefix, quant="", fused=True):
    p = P.medusa_attention_plan(m, B, max_prefix, quant, fused)
    return p["kernel"], p["queries"], p["splits"]


def test_kernels():
    assert _plan(_model(4, head_dim=64, dtype="fp32"), 1, 100) == ("portable", 1, 1)
    assert _plan(_model(32), 1, 1024) == ("tree", 32, 3)
    assert _plan(_model(32), 1, 16384) == ("tree", 64, 6)
    assert _plan(_model(32), 1, 16384, fused=False) == ("tree", 64, 16)
    assert _plan(_model(32, tree="tree15"), 1, 1024) == ("tree", 32, 5)
    assert _plan(_model(32, tree="tree1"), 1, 1024) == ("one_mfma", 1, 4)
    assert _plan(_model(32, tree="tree1"), 64, 100) == ("one_fma", 1, 1)
    assert not P.medusa_attention_plan(_model(32), 16, 1500)["ordered"] and P.medusa_attention_plan(_model(32), 16, 2560)["ordered"]


def test_errors():
    for args in [(_model(32), 0, 100), (_model(32), 1, -1), (_model(32, tree="tree15"), 1, 100, "fp8e4m3"),
                 (_model(4, head_dim=64), 1, 100, "fp8e4m3"), (_model(32, 5), 1, 100)]:
        with pytest.raises(P.MedusaError):
            P.medusa_attention_plan(*args)


@pytest.mark.parametrize("n_heads,kv_heads", [(16, 0), (32, 0), (40, 0), (32, 8)])
def test_8bit_rows_of_several_sequences_take_32_queries(n_heads, kv_heads):
    for B in range(2, 256 // n_heads + 1):
        for max_prefix in (300, 4900, 4930, 6600, 8200, 9900, 12400, 14335, 14336, 22000):
            assert _plan(_model(n_heads, kv_heads), B, max_prefix, "fp8e4m3")[:2] == ("tree", 32), (B, max_prefix)


def test_one_split_of_grouped_heads_takes_32_queries():
    for B in (5, 6, 7, 8):
        for max_prefix in (1000, 3052, 3583):
            assert _plan(_model(32, 8), B, max_prefix) == ("tree", 32, 1), (B, max_prefix)


@pytest.mark.parametrize("n_heads,B,max_prefix,kernel,splits", [
    (32, 3, 1119, "one_mfma", 3), (32, 3, 1120, "one_fma", 6), (32, 3, 2064, "one_fma", 6), (32, 5, 1364, "one_fma", 4),
    (32, 8, 564, "one_mfma", 1), (32, 8, 964, "one_fma", 3), (40, 2, 1664, "one_fma", 7), (40, 4, 1164, "one_fma", 4),
    (16, 2, 14064, "one_fma", 17), (16, 3, 4564, "one_fma", 11), (16, 12, 964, "one_fma", 3),
    (40, 1, 3583, "one_mfma", 6), (40, 1, 3584, "one_fma", 13), (16, 1, 1364, "one_mfma", 6), (32, 1, 14064, "one_mfma", 8)])
def test_single_query_splits_of_8bit_rows(n_heads, B, max_prefix, kernel, splits):
    """As many as the conversions pay for; the workspace holds them (it is sized before the row type is known)."""
    m = _model(n_heads, tree="tree1")
    assert _plan(m, B, max_prefix, "fp8e4m3") == (kernel, 1, splits)
    scratch = (B * n_heads * splits * 130 * 4 + 255) // 256 * 256
    assert P.medusa_workspace_bytes(m, B, max_prefix) - P.medusa_workspace_bytes(m, B, 0) >= scratch * (splits > 1)


@pytest.mark.parametrize("B,max_prefix,quant,splits", [
    (17, 2303, "", 1), (17, 2304, "", 4), (18, 4064, "", 4), (20, 4064, "", 1), (20, 4096, "", 4), (16, 4064, "", 2), (8, 4064, "", 4),
    (17, 2111, "fp8e4m3", 1), (17, 2112, "fp8e4m3", 4), (24, 2303, "fp8e4m3", 1), (24, 2304, "fp8e4m3", 3), (28, 3064, "fp8e4m3", 1), (28, 3072, "fp8e4m3", 3),
    (32, 4064, "fp8e4m3", 2), (12, 3583, "fp8e4m3", 2), (12, 3584, "fp8e4m3", 6), (14, 4064, "fp8e4m3", 5), (16, 3584, "fp8e4m3", 4),
    (1, 1503, "", 4), (1, 1504, "", 7), (1, 2064, "", 8), (1, 12064, "", 13), (3, 8064, "", 8), (4, 6064, "", 8), (5, 12064, "", 8), (7, 6064, "fp8e4m3", 8),
    (40, 2047, "", 1), (40, 2048, "", 2)])
def test_single_query_splits_of_grouped_heads(B, max_prefix, quant, splits):
    assert _plan(_model(32, 8, tree="tree1"), B, max_prefix, quant) == ("one_mfma", 1, splits)


@pytest.mark.parametrize("n_heads,B,max_prefix,kernel,splits", [
    (32, 2, 1791, "one_mfma", 4), (32, 2, 1792, "one_fma", 9), (32, 3, 1119, "one_mfma", 3), (32, 3, 1120, "one_fma", 6), (32, 5, 764, "one_fma", 4),
    (32, 6, 564, "one_fma", 3), (32, 8, 639, "one_mfma", 1), (32, 8, 640, "one_fma", 3), (40, 3, 1164, "one_fma", 5), (16, 3, 4064, "one_fma", 11),
    (16, 2, 6064, "one_mfma", 7), (16, 10, 764, "one_fma", 4), (32, 1, 9064, "one_mfma", 6), (40, 1, 9064, "one_mfma", 4)])
def test_single_query_splits_of_16bit_rows(n_heads, B, max_prefix, kernel, splits):
    assert _plan(_model(n_heads, tree="tree1"), B, max_prefix) == (kernel, 1, splits)


@pytest.mark.parametrize("n_heads,kv_heads,B,max_prefix,splits", [
    (32, 0, 1, 14064, 6), (32, 8, 1, 14064, 8), (16, 0, 1, 9064, 6), (16, 0, 1, 9216, 7), (16, 0, 1, 14064, 8), (16, 0, 2, 14064, 7), (16, 0, 3, 2559, 4),
    (16, 0, 3, 4564, 5), (16, 0, 4, 4564, 4), (32, 0, 2, 4095, 4), (32, 0, 2, 4564, 6), (16, 0, 5, 2559, 4), (16, 0, 5, 2560, 3), (40, 0, 2, 4564, 3),
    (32, 0, 3, 4564, 4), (16, 0, 6, 4564, 4), (16, 0, 7, 4564, 2), (16, 0, 1, 200, 1), (40, 0, 1, 7064, 6)])
def test_splits_of_the_15_node_tree(n_heads, kv_heads, B, max_prefix, splits):
    assert _plan(_model(n_heads, kv_heads, "tree15"), B, max_prefix) == ("tree", 32, splits)


def test_splits_of_48_pairs():
    """(288 workgroups of 32 queries where the launch takes the longest sequences first)"""
    assert [_plan(_model(16), 3, n) for n in (1400, 1535, 1536, 2047, 2048)] == [("tree", 32, 2)] * 2 + [("tree", 32, 3)] * 3


@pytest.mark.parametrize("tree", ["tree15", "tree64", "tree1"])
@pytest.mark.parametrize("n_heads,kv_heads", [(1, 0), (2, 0), (5, 0), (16, 0), (32, 0), (32, 8), (40, 0), (48, 12), (64, 0), (80, 0)])
def test_a_workspace_serves_shorter_prefixes_and_both_row_types(tree, n_heads, kv_heads):
    m = _model(n_heads, kv_heads, tree)
    T = P.medusa_tree_info(P.TREES[tree])["T"]
    row = 130 if tree == "tree1" else T * 130  # floats of one split's partial output and its two statistics
    for B in (1, 2, 3, 4, 5, 7, 9, 17, 40):
        base, before = P.medusa_workspace_bytes(m, B, 0), 0
        for max_prefix in sorted(list(range(0, 6000, 61)) + [2559, 2560, 3583, 3584, 4095, 4096] + list(range(6000, 40000, 977))):
            ws = P.medusa_workspace_bytes(m, B, max_prefix)
            assert ws >= before, (B, max_prefix)
            before = ws
            for quant in ("",) if tree == "tree15" else ("", "fp8e4m3"):
                for fused in (True, False):
                    splits = _plan(m, B, max_prefix, quant, fused)[2]
                    assert splits == 1 or ws - base >= B * n_heads * splits * row * 4, (B, max_prefix, quant, fused)


@pytest.mark.parametrize("max_prefix,quant,plan", [
    (8064, "", (32, 4)), (11718, "", (32, 4)), (11719, "", (64, 8)), (13564, "", (64, 8)), (12543, "fp8e4m3", (32, 4)), (12544, "fp8e4m3", (32, 8)),
    (20064, "fp8e4m3", (32, 8))])
def test_one_long_sequence_of_grouped_heads_takes_eight_splits(max_prefix, quant, plan):
    assert _plan(_model(32, 8), 1, max_prefix, quant)[1:] == plan
