"""Products of more than 64 rows whose operands do not start on 16 bytes (hidden_out and packed weights are the caller's buffers and
the interface asks for no alignment): they stay on the many-row kernel and give what aligned operands give.  Bounds: logits
against float64 on the same 16-bit operands, fp32 sums (1e-5 of the output scale); layers as in the parity tests."""
import pytest
import torch

import paper_2603_03383_amd as P
import workload as W
from tests import gpu_util as G
from tests.test_gpu_parity import TOL, _i32

pytestmark = pytest.mark.gpu


def _w(tree, dtype="bf16", **kw):
    return W.CONFIGS["cfg2_layer_bf16"].with_(**{**dict(d=256, n_heads=2, head_dim=128, ffn=704, dtype=dtype, tree=tree,
                                                        name=f"unaligned_{tree.name}"), **kw})


def _shifted(t, nbytes):
    """The same values in a buffer that starts nbytes behind a 256-byte boundary."""
    raw = torch.empty(t.numel() * t.element_size() + 256, dtype=torch.uint8, device=t.device)
    out = raw[nbytes:nbytes + t.numel() * t.element_size()]
    out.copy_(t.reshape(-1).view(torch.uint8))
    return out.view(t.dtype).view(t.shape) if nbytes % t.element_size() == 0 else out


def _families(run):
    P.medusa_profile_begin(1000)
    run()
    torch.cuda.synchronize()
    return set(P.medusa_profile_end())


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("tree,batch,vocab", [(W.TREE15, 6, 4000), (W.TREE1, 65, 96), (W.TREE64, 16, 20000)],
                         ids=lambda v: getattr(v, "name", v))
@pytest.mark.parametrize("want_logits", [True, False])
def test_lm_head_on_an_unaligned_hidden_out(dtype, tree, batch, vocab, want_logits):
    w = _w(tree, dtype, vocab=vocab)
    dm = G.device_model(w, heads=False, n_layers=1)
    T = dm.tree_info["T"]
    tokens = W.random_tokens(w, "unaligned", (batch, T)).to(torch.int32).to(G.DEV)
    seq_len = _i32([b % 3 for b in range(batch)])
    kv = P.DeviceKV(dm, batch=batch, cap=2 + T)
    buf = P.StepBuffers(dm, batch, 2, want_logits=want_logits)
    buf.hidden = _shifted(buf.hidden, 2)
    assert buf.hidden.data_ptr() % 16 == 2
    families = _families(lambda: P.tree_verify_step(dm.desc, dm.weights, tokens, kv.desc, seq_len, batch, 2, buf.node_argmax, buf.hidden,
                                                    buf.logits, buf.ws))
    assert "gemm_portable" not in families
    ref = buf.hidden.reshape(batch * T, w.d).double() @ W.lm_head(w, G.DEV).double().T
    tol = 1e-5 * max(1.0, float(ref.abs().max()))
    best = ref.gather(1, buf.node_argmax.reshape(-1, 1).long())[:, 0]
    assert float((ref.max(dim=1).values - best).max()) <= 2 * tol
    if want_logits:
        logits = buf.logits.reshape(batch * T, vocab)
        assert float((logits - ref).abs().max()) <= tol
        assert torch.equal(buf.node_argmax.reshape(-1), logits.argmax(dim=1).int())


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("tree,batch", [(W.TREE1, 65), (W.TREE15, 6), (W.TREE15, 13), (W.TREE64, 5)], ids=lambda v: getattr(v, "name", v))
@pytest.mark.parametrize("shape", [dict(), dict(d=320, n_heads=5, head_dim=64, ffn=64), dict(d=2048, n_heads=16, ffn=5632)], ids=str)
def test_layer_on_unaligned_weights(dtype, tree, batch, shape):
    _check_layer_on_unaligned_weights(_w(tree, dtype, **shape), batch)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("tree,batch,tile_rows", [(W.TREE1, 65, 96), (W.TREE15, 6, 96), (W.TREE1, 129, 192), (W.TREE64, 3, 192)],
                         ids=lambda v: getattr(v, "name", v))
def test_layer_on_unaligned_weights_in_tiles_of_96_columns(dtype, tree, batch, tile_rows):
    """The gate/up product (22016 columns) with its mixed gate and up columns, gathered into registers."""
    w = _w(tree, dtype, ffn=11008)
    plan = P.medusa_gemm_many_rows_plan(P.DTYPES[dtype], batch * P.medusa_tree_info(P.TREES[tree.name])["T"], 2 * w.ffn, w.d, 1, True)
    assert (plan["tile_rows"], plan["tile_cols"]) == (tile_rows, 96)
    _check_layer_on_unaligned_weights(w, batch)


def _check_layer_on_unaligned_weights(w, batch):
    tree, dtype = w.tree, w.dtype
    dm = G.device_model(w.with_(vocab=64), heads=False, n_layers=1)
    T = dm.tree_info["T"]
    lw = dm.layer(0)
    sizes = dict(wqkv=3 * w.d * w.d, wo=w.d * w.d, wgateup=2 * w.ffn * w.d, wdown=w.d * w.ffn)
    by_ptr = {t.data_ptr(): t for t in dm._keep}
    moved, keep = P.LayerWeights(g_attn=lw.g_attn, g_ffn=lw.g_ffn), []
    for i, name in enumerate(sizes):
        keep.append(_shifted(by_ptr[getattr(lw, name)], (2, 8, 14, 6)[i]))
        setattr(moved, name, keep[-1].data_ptr())
    seq_len = _i32([(7 * b) % 40 for b in range(batch)])
    out = []
    for weights in (lw, moved):
        kv = P.DeviceKV(dm, batch=batch, cap=40 + T, n_layers=1)
        for b in range(batch):
            kv.write(0, b, 0, *W.prefix_kv(w.with_(prefix=(40,) * batch), 0, b, G.DEV))
        x = W.hidden_state(w, "unaligned_x", batch * T, device=G.DEV).float()
        ws = dm.workspace(batch, 40)
        families = _families(lambda: P.tree_verify_layer(dm.desc, weights, 0, x, kv.desc, seq_len, batch, 40, ws))
        assert "gemm_portable" not in families
        out.append(x)
    assert torch.isfinite(out[0]).all()
    assert float((out[0] - out[1]).abs().max()) <= TOL[dtype] * max(1.0, float(out[0].abs().max()))
