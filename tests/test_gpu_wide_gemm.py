"""Products of several hundred rows that take the 192 / 256 x 256 tiles (gemm_wide.hip): row counts around the tiles' edges, one and
several bands of columns per workgroup, a last band of 96 columns, a contraction that is no whole number of packed stages, the
SwiGLU epilogue with both row tiles, the K split.  Bounds: a product against float64 on the same 16-bit operands, fp32
accumulation over ~2000 terms (1e-5 of the output scale); layers as in the parity tests.
Which kernel takes a product is the library's choice by two modelled times; every case asserts the one it is written for."""
import pytest
import torch

import paper_2603_03383_amd as P
import workload as W
from tests import gpu_util as G
from tests.test_gpu_parity import _check_layer, _i32, _layer_case

pytestmark = pytest.mark.gpu


def _plan(w, rows, N, K, max_split, swiglu=False):
    p = P.medusa_gemm_many_rows_plan(P.DTYPES[w.dtype], rows, N, K, max_split, swiglu)
    return (p["tile_rows"], p["k_splits"]) if p["wide"] else "gemm_tile"


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("tree,batch,vocab,tile_rows", [(W.TREE15, 13, 40032, 256), (W.TREE1, 257, 20000, 192), (W.TREE15, 18, 32000, 192),
                                                        (W.TREE1, 400, 40032, 192), (W.TREE64, 7, 32000, 256),
                                                        (W.TREE64, 16, 20000, 192), (W.TREE64, 16, 40032, 256)],
                         ids=lambda v: getattr(v, "name", v))
def test_lm_head_logits(dtype, tree, batch, vocab, tile_rows):
    """d 2112: 33 rounds of 64 features, 8.25 packed stages; 40032 columns: 156 bands of 256 and one of 96."""
    w = W.CONFIGS["cfg2_layer_bf16"].with_(d=2112, n_heads=33, head_dim=64, ffn=64, vocab=vocab, dtype=dtype, tree=tree,
                                           prefix=tuple(b % 3 for b in range(batch)), name=f"wide_lm{vocab}")
    dm = G.device_model(w, heads=False)
    T = dm.tree_info["T"]
    assert _plan(w, batch * T, vocab, w.d, 1) == (tile_rows, 1)
    kv = P.DeviceKV(dm, batch=batch, cap=2 + T)
    buf = P.StepBuffers(dm, batch, 2, want_logits=True)
    buf.tree_tokens.copy_(W.random_tokens(w, "wide_lm", (batch, T)).to(torch.int32))
    P.run_step(dm, kv, buf, None, None, None, _i32(list(w.prefix)), with_heads=False)
    torch.cuda.synchronize()
    hid, lm = buf.hidden.reshape(batch * T, w.d).double(), W.lm_head(w, G.DEV).double()
    logits = buf.logits.reshape(batch * T, vocab)
    for r in range(0, batch * T, 256):
        ref = hid[r:r + 256] @ lm.T
        assert (logits[r:r + 256] - ref).abs().max() <= 1e-5 * max(1.0, float(ref.abs().max())), r
    assert torch.equal(logits.gather(1, buf.node_argmax.reshape(-1, 1).long())[:, 0], logits.max(dim=1).values)


@pytest.mark.parametrize("tree,batch,vocab", [(W.TREE15, 18, 40032), (W.TREE1, 400, 40032), (W.TREE64, 16, 20000), (W.TREE64, 16, 40032)],
                         ids=lambda v: getattr(v, "name", v))
def test_argmax_without_logits(tree, batch, vocab):
    """The pass that keeps each row's best column itself gives the argmax of the pass that writes the logits, bit for bit; every
    vocabulary row exists three times (the first of equal maxima wins), in other lanes, tiles and workgroups."""
    w = W.CONFIGS["cfg2_layer_bf16"].with_(d=2112, n_heads=33, head_dim=64, ffn=64, vocab=vocab, tree=tree,
                                           prefix=tuple(b % 3 for b in range(batch)), name=f"wide_argmax{vocab}")
    dm = G.device_model(w, heads=False)
    lm = W.lm_head(w, G.DEV)
    third = vocab // 3
    perm = torch.randperm(third, generator=torch.Generator().manual_seed(3)).to(G.DEV)
    lm[third:2 * third], lm[2 * third:3 * third] = lm[:third][perm], lm[:third].flip(0)
    dm.set_lm_head(lm)
    dm.finalize()
    T = dm.tree_info["T"]
    assert _plan(w, batch * T, vocab, w.d, 1) != "gemm_tile"
    found = []
    for want in (True, False):
        kv = P.DeviceKV(dm, batch=batch, cap=2 + T)
        buf = P.StepBuffers(dm, batch, 2, want_logits=want)
        buf.tree_tokens.copy_(W.random_tokens(w, "wide_argmax", (batch, T)).to(torch.int32))
        buf.node_argmax.fill_(-7)
        buf.ws.fill_(0xA5)
        P.run_step(dm, kv, buf, None, None, None, _i32(list(w.prefix)), with_heads=False)
        torch.cuda.synchronize()
        if not want:  # the room for logits in the workspace was not written
            assert int((buf.ws == 0xA5).sum()) >= batch * T * vocab * 4
        found.append(buf.node_argmax.clone())
        if want:
            logits = buf.logits.reshape(batch * T, vocab)
            ties = (logits == logits.max(dim=1, keepdim=True).values)
            assert int((ties.sum(dim=1) >= 3).sum()) >= batch * T * 9 // 10  # (up to two rows at the end exist only once)
            assert torch.equal(buf.node_argmax.reshape(-1).long(), ties.to(torch.uint8).argmax(dim=1))
    assert torch.equal(found[0], found[1])


@pytest.mark.parametrize("dtype,d,n_heads,ffn,tree,batch,qkv,gateup", [
    # gate/up: 32 bands and one of 64 columns, 192-row tiles
    ("bf16", 2048, 16, 4128, W.TREE64, 16, "gemm_tile", (192, 1)),
    # gate/up: 44 bands, 256-row tiles
    ("fp16", 2048, 16, 5632, W.TREE64, 16, "gemm_tile", (256, 1)),
    # QKV with K in two parts, gate/up over 320 rows
    ("bf16", 4096, 32, 11008, W.TREE64, 5, (192, 2), (192, 1)),
    # 1005 rows: QKV in whole bands, gate/up in two bands per workgroup
    ("bf16", 4096, 32, 11008, W.TREE15, 67, (256, 1), (256, 1)),
])
def test_layer(dtype, d, n_heads, ffn, tree, batch, qkv, gateup):
    w = W.CONFIGS["cfg2_layer_bf16"].with_(d=d, n_heads=n_heads, ffn=ffn, dtype=dtype, tree=tree, name=f"wide_layer_{ffn}")
    rows = batch * P.medusa_tree_info(P.TREES[tree.name])["T"]
    assert _plan(w, rows, 3 * d, d, 12) == qkv and _plan(w, rows, 2 * ffn, d, 1, True) == gateup
    S_list = [(5 * b + 2) % 30 for b in range(batch)]
    _check_layer(_layer_case(w, S_list, 30, x_seed=f"wide_x{batch}"), S_list, dtype)
