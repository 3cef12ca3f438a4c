"""A node's rotated K row is the same number whichever tree attention kernel writes it (15 nodes; 64 nodes with 32 or 64 queries per
workgroup; one or several query heads per key/value head): all round the same one of a rotation's two products first.  The K
projection gives whole numbers, exact in any order of summation, chosen per rotary pair so that the products nearly cancel at the
position of one node: there the other rounding order shows in the 16-bit row."""
import numpy as np
import pytest
import torch

import paper_2603_03383_amd as P
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

S, HD, BASE, D = 300, 128, 10000.0, 1024


def _near_cancelling(pos, high):
    """Whole x, y (up to 256: exact in both types) per rotary pair, with y c + x s (high) or x c - y s near zero at `pos`."""
    angle = pos * BASE ** (-np.arange(HD // 2) / (HD // 2))
    c, s = np.cos(angle)[:, None, None], np.sin(angle)[:, None, None]
    n = np.arange(1.0, 257.0)
    x, y = n[None, :, None], n[None, None, :]
    flip = np.where(s * c > 0, -1.0, 1.0) if high else np.where(s * c > 0, 1.0, -1.0)
    r = np.abs((flip * y) * c + x * s) if high else np.abs(x * c - (flip * y) * s)
    best = (r / (x + y)).reshape(HD // 2, -1).argmin(1)
    return n[best // 256], flip[:, 0, 0] * n[best % 256]


def _k_rows(tree, dtype, wk, kv_heads, max_prefix):
    td = {"bf16": torch.bfloat16, "fp16": torch.float16}[dtype]
    dm = P.DeviceModel(d=D, n_heads=D // HD, head_dim=HD, ffn=704, vocab=32, n_layers=1, dtype=dtype, tree=tree, n_kv_heads=kv_heads,
                       rope_base=BASE, device=G.DEV)
    zero = lambda *s: torch.zeros(*s, dtype=td)  # noqa: E731
    one = torch.ones(D, dtype=td)
    dm.add_layer(zero(D, D), wk.to(td), wk.to(td), zero(D, D), zero(704, D), zero(704, D), zero(D, 704), one, one)
    dm.finalize()
    T = dm.tree_info["T"]
    assert P.medusa_attention_plan(dm.desc, 1, max_prefix)["queries"] == (64 if max_prefix > 512 else 32)
    kv = P.DeviceKV(dm, 1, max_prefix + T)
    x = torch.ones(T, D, dtype=torch.float32, device=G.DEV)
    P.tree_verify_layer(dm.desc, dm.layer(0), 0, x, kv.desc, torch.tensor([S], dtype=torch.int32, device=G.DEV), 1, max_prefix,
                        dm.workspace(1, max_prefix))
    k, v = kv.read(0, 0, S, T)
    torch.cuda.synchronize()
    assert torch.equal(v.cpu().float(), wk[:, 0].view(kv_heads, 1, HD).expand(kv_heads, T, HD))  # the sums are exact
    return k.cpu()


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("kv_heads", [8, 4])
def test_k_row_does_not_depend_on_the_kernel(dtype, kv_heads):
    wk = torch.zeros(kv_heads * HD, D)
    for h in range(kv_heads):
        x, y = _near_cancelling(S + h % 4, high=h // 4 == 0 if kv_heads == 8 else h % 2 == 0)
        wk[h * HD:h * HD + 64, 0], wk[h * HD + 64:(h + 1) * HD, 0] = torch.from_numpy(x), torch.from_numpy(y)
    node_at = {t: [P.medusa_tree_tables(P.TREES[t])["depth"].tolist().index(e) for e in range(4)] for t in ("tree15", "tree64")}
    ref = _k_rows("tree64", dtype, wk, kv_heads, 512)[:, node_at["tree64"]]
    wide = _k_rows("tree64", dtype, wk, kv_heads, 60000)[:, node_at["tree64"]]
    small = _k_rows("tree15", dtype, wk, kv_heads, 512)[:, node_at["tree15"]]
    assert torch.equal(ref, wide), int((ref != wide).sum())
    assert torch.equal(ref, small), int((ref != small).sum())
