"""The tree's own K and V rows in the fused tree attention: they enter the product from LDS and reach the cache, whose 1 KiB units
may also hold prefix keys or slots behind the tree.  Lengths that put the first and last tree slot on every kind of place in
a block of 32 keys; sequences beside each other; more partial-sum slots than are requested together (narrow models); grouped heads
(one workgroup of a group writes); both numbers of queries per workgroup.  Output, tree rows and the untouched prefix rows are
checked; bounds: the layer parity tests'.  Slots behind the tree keep their bytes, also those that another stream writes during the
pass."""
import pytest
import torch

import paper_2603_03383_amd as P
import workload as W
from tests import gpu_util as G
from tests.test_gpu_kv8 import check_layer_kv8
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 3, 4, 15, 17, 31, 32, 33, 49, 63, 97]


def _w(tree, dtype="bf16", n_heads=4, **kw):
    return W.CONFIGS["cfg2_layer_bf16"].with_(d=128 * n_heads, n_heads=n_heads, head_dim=128, ffn=704, dtype=dtype, tree=tree,
                                              name=f"rows_{tree.name}_{n_heads}", **kw)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("tree", [W.TREE15, W.TREE64], ids=lambda t: t.name)
@pytest.mark.parametrize("n_heads,kv_heads", [(4, 0), (8, 2)])
def test_layer_rows_at_block_edges(tree, dtype, n_heads, kv_heads):
    w = _w(tree, dtype, n_heads, n_kv_heads=kv_heads)
    for S in EDGES:
        _check_layer(_layer_case(w, [S], 97, x_seed=f"rows_x{S}"), [S], dtype)
    _check_layer(_layer_case(w, EDGES, 97, x_seed="rows_xb"), EDGES, dtype)


@pytest.mark.parametrize("max_prefix,queries", [(97, 32), (118500, 64)])
def test_layer_rows_at_block_edges_8bit(max_prefix, queries):
    w = _w(W.TREE64, kv_quant="fp8e4m3")
    assert G.attention_plan(w, 1, max_prefix)["queries"] == queries
    for S in (0, 1, 15, 31, 33, 63):
        check_layer_kv8(_layer_case(w.with_(prefix=(S,)), [S], max_prefix, x_seed=f"rows8_x{S}"), [S], w.with_(prefix=(S,)), f"rows8_x{S}")


def test_layer_rows_with_64_queries_per_workgroup():
    w = _w(W.TREE64)
    assert G.attention_plan(w, 1, 47000)["queries"] == 64
    for S in (0, 17, 33):
        _check_layer(_layer_case(w, [S], 47000, x_seed=f"rows64_x{S}"), [S], "bf16")


def test_the_narrow_models_have_more_slots_than_are_requested_together():
    assert P.medusa_gemm_plan(P.MDZ_BF16, 64, 3 * 512, 512, 12)["max_slots"] > 2


FORMATS = [(W.TREE15, "bf16", ""), (W.TREE64, "bf16", ""), (W.TREE64, "fp16", ""), (W.TREE64, "bf16", "fp8e4m3")]


def _pass_over_a_full_cache(tree, dtype, quant, max_prefix, kv_heads=2, n_heads=4, behind=40):
    """A layer call over one sequence per length of EDGES, every slot of the cache holding a row; and those rows as read back."""
    w = _w(tree, dtype, n_heads, n_kv_heads=kv_heads)
    dm = G.device_model(w.with_(vocab=64), heads=False, n_layers=1)
    T, B = dm.tree_info["T"], len(EDGES)
    cap = max_prefix + T + behind
    kv = P.DeviceKV(dm, B, cap, n_layers=1, quant=quant)
    gen = torch.Generator(G.DEV).manual_seed(5)
    rows = lambda n: torch.empty(kv_heads, n, 128, device=G.DEV).normal_(generator=gen).to(dm.tdtype)  # noqa: E731
    for b in range(B):
        kv.write(0, b, 0, rows(cap), rows(cap))
    before = [kv.read(0, b, 0, cap) for b in range(B)]
    x = W.hidden_state(w, "full_x", B * T, device=G.DEV).float()
    lens = torch.tensor(EDGES, dtype=torch.int32, device=G.DEV)
    ws = dm.workspace(B, max_prefix)

    def run():
        P.tree_verify_layer(dm.desc, dm.layer(0), 0, x.clone(), kv.desc, lens, B, max_prefix, ws)
    return kv, T, before, run, rows


@pytest.mark.parametrize("queries", [32, 64])
@pytest.mark.parametrize("tree,dtype,quant", FORMATS, ids=lambda v: getattr(v, "name", v))
def test_slots_outside_the_tree_keep_their_bytes(tree, dtype, quant, queries):
    """64 queries per workgroup: five key-splits of a long prefix; with 8-bit rows one split of more heads than CUs."""
    n_heads, max_prefix = (4, 97) if queries == 32 else (24, 97) if quant else (4, 17000)
    kv, T, before, run, _ = _pass_over_a_full_cache(tree, dtype, quant, max_prefix, n_heads=n_heads)
    assert T == 15 or P.medusa_attention_plan(kv.model.desc, len(EDGES), max_prefix, quant)["queries"] == queries
    run()
    torch.cuda.synchronize()
    for b, S in enumerate(EDGES):
        for old, new in zip(before[b], kv.read(0, b, 0, before[b][0].shape[1])):
            assert torch.equal(old[:, :S], new[:, :S]) and torch.equal(old[:, S + T:], new[:, S + T:])
            assert not torch.equal(old[:, S:S + T], new[:, S:S + T])


@pytest.mark.parametrize("tree,dtype,quant", FORMATS, ids=lambda v: getattr(v, "name", v))
def test_rows_written_behind_the_tree_during_a_pass_stay(tree, dtype, quant):
    behind = 40
    kv, T, before, run, rows = _pass_over_a_full_cache(tree, dtype, quant, 97, behind=behind)
    run()
    torch.cuda.synchronize()
    tree_rows = [[t.clone() for t in kv.read(0, b, S, T)] for b, S in enumerate(EDGES)]
    side = torch.cuda.Stream()
    kept = []
    for _ in range(4):
        new = [(rows(behind), rows(behind)) for _ in EDGES]
        kept.append(new)
        torch.cuda.synchronize()
        for i in range(6):
            run()
            with torch.cuda.stream(side):
                for b, S in enumerate(EDGES[2 * i:2 * i + 2], 2 * i):
                    P.medusa_kv_write(kv.desc, 0, b, S + T, behind, *new[b])
        torch.cuda.synchronize()
        ref = P.DeviceKV(kv.model, len(EDGES), behind, n_layers=1, quant=quant)
        for b, S in enumerate(EDGES):
            ref.write(0, b, 0, *new[b])
            for got, want in zip(kv.read(0, b, S + T, behind), ref.read(0, b, 0, behind)):
                assert torch.equal(got, want)
            for got, want in zip(kv.read(0, b, S, T), tree_rows[b]):
                assert torch.equal(got, want)
            for got, want in zip(kv.read(0, b, 0, S + T), before[b]):
                assert torch.equal(got[:, :S], want[:, :S])
