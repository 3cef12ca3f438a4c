"""The softmax weights of the single-query attention and of the 15-node tree are fp32 numbers: products with V lose nothing against
fp32.  A layer in which everything around the attention is exact makes its output visible: x is +-1 (its norm is then +-1 in
both 16-bit types), every row of Wq, Wk, Wv has ONE nonzero entry, the rotary base is so large that the features in use do not
turn, Wo is 1024 x identity and the feed-forward block adds zero.  So (x_out - x) / 1024 is the attention's 16-bit output.

Bound against float64: half a unit in the last place of the 16-bit output (2^-8 |att| in bf16, 2^-11 |att| in fp16; 2^-25 where
binary16 is subnormal) plus 3e-6 of the largest value row, about ten times what fp32 scores and sums leave (a score of 64 fp32
products is off by ~3e-7).  Weights rounded to 16 bits leave 2^-8 / 2^-11 each, i.e. 1e-4 .. 1e-3 / 2e-5 .. 1e-4 of the value rows."""
import numpy as np
import pytest
import torch

import paper_2603_03383_amd as P
import workload as W
from oracle import kv8
from oracle import medusa as O
from oracle import tree as OT

pytestmark = pytest.mark.gpu

HD, OUT = 128, 1024.0
TREES = {"tree1": W.TREE1, "tree15": W.TREE15}
ACTIVE = np.r_[32:64, 96:128]  # features whose rotary angle is below 1e-15 at every position used here


def _one_entry_rows(rng, n, d, std, dtype, active=None):
    """[n, d] with one nonzero per row (so a product with +-1 is exact); rows of inactive features stay zero."""
    w = np.zeros((n, d))
    val = O.round_to_storage(rng.normal(0.0, std, n), dtype)
    if active is not None:
        val[~np.isin(np.arange(n) % HD, active)] = 0.0
    w[np.arange(n), rng.integers(0, d, n)] = val
    return w


def _attention(tree_name, dtype, n_heads, kv_heads, S_list, max_prefix, quant="", v_std=1.0):
    """(attention output of the layer [B, T, n_heads, 128], the same in float64, largest |V|)"""
    rng = np.random.default_rng(7)
    tw = TREES[tree_name]
    tree = OT.build_tree(tw.caps, tw.budgets)
    T, B, d, ffn = tree["T"], len(S_list), n_heads * HD, 64
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a))  # noqa: E731
    dm = P.DeviceModel(d=d, n_heads=n_heads, head_dim=HD, ffn=ffn, vocab=64, n_layers=1, dtype=dtype, tree=tree_name,
                       n_kv_heads=kv_heads, rope_base=1e38)
    wq = _one_entry_rows(rng, d, d, 1.0, dtype, ACTIVE)
    wk = _one_entry_rows(rng, kv_heads * HD, d, 1.0, dtype, ACTIVE)
    wv = _one_entry_rows(rng, kv_heads * HD, d, v_std, dtype)
    zeros = np.zeros((ffn, d))
    dm.add_layer(t(wq), t(wk), t(wv), t(OUT * np.eye(d)), t(zeros), t(zeros), t(np.zeros((d, ffn))), t(np.ones(d)), t(np.ones(d)))
    dm.finalize()
    kv = P.DeviceKV(dm, batch=B, cap=max_prefix + T, quant=quant)
    x = rng.choice([-1.0, 1.0], (B * T, d))
    rows = (lambda a: kv8.roundtrip_rows(a)) if quant else (lambda a: O.round_to_storage(a, dtype))
    ref, v_max = np.zeros((B, T, n_heads, HD)), 0.0
    for b, S in enumerate(S_list):
        k = O.round_to_storage(rng.normal(0.0, 1.0, (kv_heads, S, HD)), dtype)
        v = O.round_to_storage(rng.normal(0.0, v_std, (kv_heads, S, HD)), dtype)
        if S:
            kv.write(0, b, 0, t(k), t(v))
        xb = x[b * T:(b + 1) * T]
        own = lambda w: (xb @ w.T).reshape(T, kv_heads, HD).transpose(1, 0, 2)  # noqa: E731
        kc, vc = rows(np.concatenate([k, own(wk)], axis=1)), rows(np.concatenate([v, own(wv)], axis=1))
        q = (xb @ wq.T).reshape(T, n_heads, HD).transpose(1, 0, 2)
        ref[b] = O._attend(q, kc, vc, O.tree_visibility(tree, S), HD).transpose(1, 0, 2)
        v_max = max(v_max, float(np.abs(vc).max()))
    xd = torch.from_numpy(x).to(torch.float32).to("cuda:0")
    P.tree_verify_layer(dm.desc, dm.layer(0), 0, xd, kv.desc, torch.tensor(S_list, dtype=torch.int32, device="cuda:0"), B, max_prefix,
                        dm.workspace(B, max_prefix))
    torch.cuda.synchronize()
    out = (xd.cpu().numpy().astype(np.float64) - x).reshape(B, T, n_heads, HD) / OUT
    return out, ref, v_max


def _check(tree, dtype, *args, **kw):
    out, ref, v_max = _attention(tree, dtype, *args, **kw)
    # (x + 1024 att is rounded to fp32 once: 2^-24 of it)
    bound = {"bf16": 2.0 ** -8, "fp16": 2.0 ** -11}[dtype] * np.abs(ref) + 3e-6 * v_max + 2.0 ** -24 * (1.0 / OUT + np.abs(ref))
    if dtype == "fp16":
        bound += 2.0 ** -25
    over = np.abs(out - ref) / bound
    print(f"{tree} {dtype} {kw}: largest error / bound {over.max():.3f}, error of outputs near zero / V "
          f"{np.abs(out - ref)[np.abs(ref) < 1e-3 * v_max].max(initial=0.0) / v_max:.2e}")
    assert over.max() <= 1.0


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("n_heads,kv_heads", [(4, 4), (8, 2)])
def test_single_query(dtype, n_heads, kv_heads):
    _check("tree1", dtype, n_heads, kv_heads, [40, 0, 5, 100, 700, 31], 700)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("v_std", [1.0, 1e-3, 1e-4])
def test_single_query_eight_bit_rows(dtype, v_std):
    """Value rows whose scales (largest entry / 448), times a weight, are far below binary16's normal range."""
    _check("tree1", dtype, 4, 2, [40, 0, 5, 100, 700, 31], 700, quant="fp8e4m3", v_std=v_std)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("n_heads,kv_heads", [(4, 4), (8, 2)])
def test_fifteen_node_tree(dtype, n_heads, kv_heads):
    _check("tree15", dtype, n_heads, kv_heads, [18, 0, 45, 600], 600)
