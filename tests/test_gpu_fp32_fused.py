"""fp32 storage: the gate/up product with the SwiGLU in its epilogue (row counts at the edges of its 16-, 32- and 64-row tiles) and the
Medusa heads' vocabulary products in one launch, with their selection in another (vocabularies below and above the two-stage
selection's threshold, several sequences, with and without root tokens).  Bounds: the fp32 parity tests'."""
import numpy as np
import pytest
import torch

import paper_2603_03383_amd as P
import workload as W
from tests import gpu_util as G
from tests.test_gpu_parity import _check_layer, _layer_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tree,batches", [(W.TREE1, [1, 16, 17, 32, 33, 64, 65]), (W.TREE15, [1, 2, 3, 5]), (W.TREE64, [1, 2])],
                         ids=["1 node", "15 nodes", "64 nodes"])
def test_layer_swiglu_rows(tree, batches):
    w = W.CONFIGS["cfg2_layer_bf16"].with_(d=128, n_heads=2, head_dim=64, ffn=176, dtype="fp32", tree=tree, name=f"f32_ffn_{tree.name}")
    for n in batches:
        S_list = [(7 * b) % 40 for b in range(n)]
        _check_layer(_layer_case(w, S_list, 40, x_seed=f"f32_ffn_x{n}"), S_list, "fp32")


@pytest.mark.parametrize("vocab", [64, 1000, 1024, 8192])
@pytest.mark.parametrize("batch,root", [(1, True), (3, True), (17, False)])
@pytest.mark.parametrize("tree", ["tree15", "tree64", "tree64k5"])
def test_heads_select_what_their_own_logits_say(tree, vocab, batch, root):
    d, dev = 128, G.DEV
    gen = torch.Generator(dev).manual_seed(vocab + batch)
    normal = lambda *s: torch.empty(*s, device=dev).normal_(0.0, 1.0, generator=gen)  # noqa: E731
    dm = P.DeviceModel(d=d, n_heads=2, head_dim=64, ffn=176, vocab=vocab, n_layers=1, dtype="fp32", tree=tree, device=dev)
    lm, topk = normal(vocab, d), dm.tree_info["topk"]
    dm.set_lm_head(lm)
    w1s, lms = [normal(d, d) for _ in topk], [normal(vocab, d) for _ in topk]
    for a, b in zip(w1s, lms):
        dm.add_medusa_head(a, None, b)
    dm.finalize()
    h = normal(batch, 1, d)
    roots = torch.arange(batch, dtype=torch.int32, device=dev) if root else None
    buf = P.StepBuffers(dm, batch, 0, want_head_logits=True)
    P.medusa_heads(dm.desc, dm.weights, h, None, roots, batch, 1, buf.cand_flat, buf.tree_tokens, buf.head_logits, buf.ws)
    torch.cuda.synchronize()
    x = h[:, 0].double()
    for b in range(batch):
        got = buf.cand_flat[b].cpu().tolist()
        rows = [x[b] @ lm.double().T] + [(x[b] + torch.nn.functional.silu(x[b] @ w1.double().T)) @ m.double().T for w1, m in zip(w1s, lms)]
        assert got[0] == (b if root else int(buf.head_logits[b, 0].argmax()))
        seg = 1
        for j, k in enumerate(topk, 1):
            own = buf.head_logits[b, j].cpu().numpy()
            ref = rows[j].cpu().numpy()
            assert np.abs(own - ref).max() <= 1e-5 * max(1.0, np.abs(ref).max())
            order = np.lexsort((np.arange(vocab), -own))[:k]      # value descending, then lower id
            assert got[seg:seg + k] == order.tolist()
            seg += k
