"""tree_verify_layer_static where the K splits that the layer prefers do not fit the built-in buffer: it runs on fewer partial sums,
and agrees with the layer on a caller workspace up to the order of fp32 sums in front of bf16 roundings (the layer bound)."""
import pytest
import torch

import paper_2603_03383_amd as P
import workload as W
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,prefix", [(10, 512), (12, 16384)])
def test_small_tree_batches_that_need_fewer_partial_sums(batch, prefix):
    w = W.CONFIGS["cfg2_layer_bf16"].with_(tree=W.TREE15, prefix=(40,) * batch)
    dm = G.device_model(w.with_(vocab=1024), heads=False, n_layers=1)
    T = dm.tree_info["T"]
    seq_len = torch.tensor([3 * b for b in range(batch)], dtype=torch.int32, device=G.DEV)
    outs = []
    for static in (False, True):
        kv = P.DeviceKV(dm, batch=batch, cap=prefix + T, n_layers=1)
        for b in range(batch):
            kv.write(0, b, 0, *W.prefix_kv(w, 0, b, G.DEV))
        x = W.hidden_state(w, "static_batch", batch * T, device=G.DEV).float()
        if static:
            P.tree_verify_layer_static(dm.desc, dm.layer(0), 0, x, kv.desc, seq_len, batch, prefix)
        else:
            P.tree_verify_layer(dm.desc, dm.layer(0), 0, x, kv.desc, seq_len, batch, prefix, dm.workspace(batch, prefix))
        torch.cuda.synchronize()
        outs.append(x)
    scale = float(outs[0].abs().max())
    assert torch.isfinite(outs[0]).all() and scale > 1.0
    assert float((outs[0] - outs[1]).abs().max()) <= 2e-2 * scale
