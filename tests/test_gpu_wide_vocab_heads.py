"""The Medusa heads' vocabulary products over at least two whole bands per workgroup and up to 32 rows (two half stages of the weights in
flight instead of three): vocabularies around the size at which that begins, with a ragged last band, at the edges of the row
range; two or three K-stages per band and two or three bands per workgroup, so that ranges have even and odd numbers of stages and a band
ends in either half of the pipeline's trips.  A row's sums do not depend on how many rows run beside it, so the logits must equal those of 33 rows, which take the other
kernel, bit for bit; and they must be close to float64 (bound: the bf16 parity tests')."""
import pytest
import torch

import paper_2603_03383_amd as P
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("heads", [2, 3])
@pytest.mark.parametrize("bands_per_cu,more", [(2, -128), (2, 0), (2, 96), (3, 0), (3, 32)])
def test_logits_equal_those_of_more_rows(bands_per_cu, more, heads, dtype):
    d, dev = 128 * heads, G.DEV
    cus = torch.cuda.get_device_properties(dev).multi_processor_count
    vocab = bands_per_cu * cus * 128 + more
    assert P.medusa_gemm_plan(P.DTYPES[dtype], 32, vocab, d, 1)["grid"] == cus  # whole bands, 2 or 3 per workgroup
    gen = torch.Generator(dev).manual_seed(vocab)
    td = {"bf16": torch.bfloat16, "fp16": torch.float16}[dtype]
    normal = lambda *s, std=1.0: torch.empty(*s, dtype=td, device=dev).normal_(0.0, std, generator=gen)  # noqa: E731
    dm = P.DeviceModel(d=d, n_heads=heads, head_dim=128, ffn=704, vocab=vocab, n_layers=1, dtype=dtype, tree="tree15", device=dev)
    dm.set_lm_head(normal(vocab, d, std=0.05))
    mats = [(normal(d, d, std=0.05), normal(vocab, d, std=0.05)) for _ in dm.tree_info["topk"]]
    for w1, lm in mats:
        dm.add_medusa_head(w1, None, lm)
    dm.finalize()
    h = normal(33, 1, d)
    logits = {}
    for rows in (33, 32, 17, 1):
        buf = P.StepBuffers(dm, rows, 0, want_head_logits=True)
        P.medusa_heads(dm.desc, dm.weights, h[:rows].contiguous(), None, torch.zeros(rows, dtype=torch.int32, device=dev), rows, 1, buf.cand_flat,
                       buf.tree_tokens, buf.head_logits, buf.ws)
        logits[rows] = buf.head_logits[:, 1:].clone()
    torch.cuda.synchronize()
    for rows in (32, 17, 1):
        assert torch.equal(logits[rows], logits[33][:rows])
    x = h[:, 0].double()
    for k, (w1, lm) in enumerate(mats):
        ref = (x + torch.nn.functional.silu(x @ w1.double().T)) @ lm.double().T
        assert (logits[33][:, k].double() - ref).abs().max() <= 2e-2 * max(1.0, float(ref.abs().max()))
