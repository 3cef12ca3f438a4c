"""More rows than 32-bit offsets into X reach: 3100 sequences on the 64-node tree, whose feed-forward activations (198400 x 11008) pass
2^32 bytes.  The layer stays on the many-row kernels, and the first, a middle and the last sequences come out as they do
alone (same values, fp32 sums in another order in front of 16-bit roundings: the layer bound)."""
import pytest
import torch

import paper_2603_03383_amd as P
import workload as W
from tests import gpu_util as G
from tests.test_gpu_parity import TOL

pytestmark = pytest.mark.gpu


def test_layer_whose_activations_pass_4_gib():
    w = W.CONFIGS["cfg2_layer_bf16"].with_(d=64, n_heads=1, head_dim=64, ffn=11008, tree=W.TREE64, name="many_sequences")
    dm = G.device_model(w.with_(vocab=64), heads=False, n_layers=1)
    T, batch = dm.tree_info["T"], 3100
    assert batch * T * w.ffn * 2 > 2 ** 32
    x_all = W.hidden_state(w, "many_x", batch * T, device=G.DEV).float().view(batch, T, w.d)

    def run(pick):
        n = len(pick)
        x = x_all[pick].reshape(n * T, w.d).contiguous()
        kv = P.DeviceKV(dm, batch=n, cap=T, n_layers=1)
        seq_len = torch.zeros(n, dtype=torch.int32, device=G.DEV)
        ws = dm.workspace(n, 0)
        P.medusa_profile_begin(100)
        P.tree_verify_layer(dm.desc, dm.layer(0), 0, x, kv.desc, seq_len, n, 0, ws)
        torch.cuda.synchronize()
        assert "gemm_portable" not in P.medusa_profile_end()
        return x.view(n, T, w.d)

    some = [0, 1, 1517, batch - 2, batch - 1]
    out, alone = run(list(range(batch)))[some], run(some)
    assert torch.isfinite(out).all() and float(out.abs().max()) > 1.0
    assert float((out - alone).abs().max()) <= TOL["bf16"] * max(1.0, float(alone.abs().max()))
