"""fp32 storage away from the tiny model's own sizes: row counts around the 16- and 64-row tiles of the GEMM, contractions of
fewer chunks than it has waves, a vocabulary that is no multiple of anything, head sizes with and without the attention's
eight-feature loads, keys beyond one of its chunks.  Bound: 1e-5 of the output scale, the fp32 bound of the parity tests."""
import numpy as np
import pytest
import torch

import paper_2603_03383_amd as P
import workload as W
from oracle import medusa as O
from tests import gpu_util as G
from tests import util as U
from tests.test_gpu_parity import TOL, _check_layer, _i32, _layer_case, _scale

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tree,batch", [(W.TREE1, 1), (W.TREE15, 1), (W.TREE1, 16), (W.TREE1, 17), (W.TREE15, 2),
                                        (W.TREE1, 33), (W.TREE64, 1), (W.TREE1, 65), (W.TREE15, 9)],
                         ids=lambda v: getattr(v, "name", v))
def test_layer_row_counts(tree, batch):
    w = W.CONFIGS["cfg1_tiny_fp32"].with_(tree=tree, n_layers=1, name=f"fp32_rows_{tree.name}_{batch}")
    S_list = [(29 * b + 3) % 80 for b in range(batch)]
    _check_layer(_layer_case(w, S_list, 80, x_seed=f"fp32_x{batch}"), S_list, "fp32")


@pytest.mark.parametrize("n_heads,head_dim,ffn,S", [(3, 16, 16, 5), (4, 20, 48, 40), (1, 256, 688, 70), (2, 64, 96, 2500)])
def test_layer_shapes(n_heads, head_dim, ffn, S):
    w = W.CONFIGS["cfg1_tiny_fp32"].with_(d=n_heads * head_dim, n_heads=n_heads, head_dim=head_dim, ffn=ffn, n_layers=1,
                                          name=f"fp32_{n_heads}x{head_dim}")
    _check_layer(_layer_case(w, [S, 0], S, x_seed=f"fp32_s{S}"), [S, 0], "fp32")


@pytest.mark.parametrize("vocab,batch", [(1003, 1), (517, 3)])
def test_step_with_an_odd_vocabulary(vocab, batch):
    w = W.CONFIGS["cfg1_tiny_fp32"].with_(vocab=vocab, prefix=tuple(20 + 7 * b for b in range(batch)), name=f"fp32_v{vocab}")
    tree, model, dm = U.oracle_tree(w), U.oracle_model(w), G.device_model(w)
    T, S_max = tree["T"], max(w.prefix)
    kv = G.device_kv_random_prefix(dm, w, cap=S_max + T)
    tokens = W.random_tokens(w, "fp32_v", (batch, T)).numpy().astype(np.int32)
    buf = P.StepBuffers(dm, batch, S_max, want_logits=True)
    buf.tree_tokens.copy_(_i32(tokens))
    P.run_step(dm, kv, buf, None, None, None, _i32(list(w.prefix)), with_heads=False)
    torch.cuda.synchronize()
    for b in range(batch):
        kc, vc = U.oracle_prefix_cache(w, b, w.prefix[b] + T)
        ref = O.tree_verify_step(tokens[b], model, kc, vc, w.prefix[b], tree)
        lg = buf.logits[b].cpu().numpy()
        assert np.abs(lg - ref["logits"]).max() <= TOL["fp32"] * _scale(ref["logits"])
        assert np.array_equal(buf.node_argmax[b].cpu().numpy(), np.argmax(lg, axis=-1))
