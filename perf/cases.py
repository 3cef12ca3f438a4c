"""The work that a user of this framework has it do, as cases that a program can time.

A case is a dict of plain values: a decoder shape, a storage type, a static tree, a batch of sequences with their prefix
lengths, and which calls of the decode loop a pass makes:

* ``step``:  tree_verify_step -> accept_longest_prefix -> kv_compact, the loop's body once the candidates are known (with
  ``heads`` also the medusa_heads call in front of it, i.e. run_step as a whole);
* ``layer``: tree_verify_layer alone;
* ``heads``: medusa_heads alone.

Weights are random with the spread of trained decoders: std 0.02, the two matrices that write to the residual stream scaled
down by sqrt(2 x layers), RMSNorm gains around 1.  The vocabulary matrices carry a planted preference (the row of one token is
correlated with what the model sees), so that argmax and top-k are decided by margins as they are in a trained model, and
every sequence's tree holds a continuation that the model accepts to some depth.
"""
import math

import torch

import paper_2603_03383_amd as P

DEV = "cuda:0"

# Decoder shapes: the 7B-class shape of the benchmark, the paper-shaped variant (grouped heads), the tiny model of the
# tests, and one narrower and one wider shape of the same family.
SHAPES = {
    "7b": dict(d=4096, n_heads=32, kv_heads=32, head_dim=128, ffn=11008, vocab=128000),
    "paper": dict(d=4096, n_heads=32, kv_heads=8, head_dim=128, ffn=12800, vocab=153600),
    "tiny": dict(d=256, n_heads=4, kv_heads=4, head_dim=64, ffn=688, vocab=1024),
    "narrow": dict(d=2048, n_heads=16, kv_heads=16, head_dim=128, ffn=5632, vocab=32000),
    "wide": dict(d=5120, n_heads=40, kv_heads=40, head_dim=128, ffn=13824, vocab=32000),
}
TREE_T = {"tree15": 15, "tree64": 64, "tree1": 1, "tree64k5": 64}
TREE_TOPK = {"tree15": (2, 2, 2), "tree64": (10, 10, 4, 4), "tree1": (), "tree64k5": (9, 10, 4, 3, 2)}


def _case(what, shape, dtype, tree, layers, batch, lo, hi, **more):
    c = dict(what=what, shape=shape, dtype=dtype, tree=tree, layers=layers, batch=batch, prefix_lo=lo, prefix_hi=hi,
             heads=False, kv8=False, ffn_f16=False, logits=True)
    c.update(more)
    return c


def listed():
    named = lambda name, *a, **k: dict(_case(*a, **k), name=name)  # noqa: E731
    return [
        # the smallest call: the tiny fp32 model's whole step (heads, 15-node verify, accept, compact), all launches and latency
        named("tiny_fp32_step", "step", "tiny", "fp32", "tree15", 2, 1, 64, 64, heads=True),
        # one decoder layer at the 7B-class shape, short prefix: the call a pipeline stage or a layer-wise host makes
        named("layer_512", "layer", "7b", "bf16", "tree64", 1, 1, 512, 512, logits=False),
        # the benchmark's headline: one 64-node verify step of the whole 32-layer model at a 1K prefix
        named("step_1k", "step", "7b", "bf16", "tree64", 32, 1, 1024, 1024),
        # the long-prefix end of the same step; as in a decode loop only tokens and the hidden state are asked for
        named("step_16k", "step", "7b", "bf16", "tree64", 32, 1, 16384, 16384, logits=False),
        # long prefix with 8-bit cache rows, an odd length
        named("step_7k_kv8", "step", "7b", "bf16", "tree64", 8, 1, 7001, 7001, kv8=True),
        # the paper-shaped model in its own precision: grouped heads, five Medusa heads
        named("paper_1k_fp16", "step", "paper", "fp16", "tree64k5", 34, 1, 1024, 1024),
        # candidate generation: four Medusa heads over a 128000-word vocabulary from one hidden state
        named("heads_b1", "heads", "7b", "bf16", "tree64", 1, 1, 0, 0),
        # autoregressive decoding (the one-node tree), the baseline that every speculative step is held against
        named("ar_1k", "step", "7b", "bf16", "tree1", 32, 1, 1024, 1024),
        # autoregressive decoding of a ragged batch of the grouped-head model
        named("ar_b24", "step", "paper", "fp16", "tree1", 8, 24, 90, 3000),
        # the small tree over a few ragged sequences: 90 rows, a size that is a multiple of nothing
        named("tree15_b6", "step", "7b", "bf16", "tree15", 8, 6, 40, 1500),
        # a few ragged sequences on the 64-node tree, binary16 feed-forward operands
        named("step_b3_ffn16", "step", "7b", "bf16", "tree64", 8, 3, 200, 2500, ffn_f16=True),
        # the ragged batch of sixteen sequences: 1024 rows, the compute-bound end
        named("ragged_b16", "step", "7b", "bf16", "tree64", 8, 16, 256, 4096, logits=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["tiny", "layer", "step", "step", "step", "batch", "batch", "ar", "ar", "heads"])
    dtype = rng.choice(["bf16", "bf16", "fp16"])
    if kind == "tiny":
        s = _log_int(rng, 8, 400)
        return _case("step", "tiny", "fp32", rng.choice(["tree15", "tree64", "tree64k5"]), rng.randint(1, 3), rng.randint(1, 3),
                     max(1, s // 2), s, heads=rng.random() < 0.7)
    if kind == "layer":
        s = _log_int(rng, 30, 12000)
        return _case("layer", rng.choice(["7b", "paper", "narrow", "wide"]), dtype, rng.choice(["tree64", "tree64", "tree15", "tree1"]),
                     1, 1, s, s, logits=False)
    if kind == "step":
        s = _log_int(rng, 60, 14000)
        shape = rng.choice(["7b", "7b", "paper", "narrow", "wide"])
        return _case("step", shape, dtype, "tree64k5" if shape == "paper" else "tree64", rng.randint(2, 12), 1, s, s,
                     kv8=rng.random() < 0.25, logits=rng.random() < 0.5, ffn_f16=dtype == "bf16" and rng.random() < 0.2)
    if kind == "batch":
        tree = rng.choice(["tree64", "tree64", "tree15"])
        hi = _log_int(rng, 200, 4000)
        return _case("step", rng.choice(["7b", "7b", "paper", "narrow"]), dtype, tree, rng.randint(1, 6), _log_int(rng, 2, 14), max(1, hi // 12),
                     hi, logits=rng.random() < 0.5)
    if kind == "ar":
        hi = _log_int(rng, 100, 6000)
        return _case("step", rng.choice(["7b", "paper", "narrow", "wide"]), dtype, "tree1", rng.randint(2, 8), _log_int(rng, 1, 100),
                     max(1, hi // 9), hi, kv8=rng.random() < 0.25, logits=rng.random() < 0.5)
    return _case("heads", rng.choice(["7b", "7b", "narrow", "wide"]), dtype, rng.choice(["tree64", "tree64", "tree15"]), 1, _log_int(rng, 1, 16),
                 0, 0)


def _prefixes(case):
    """Prefix lengths of the batch: spread evenly over [lo, hi], in a scattered order."""
    n, lo, hi = case["batch"], case["prefix_lo"], case["prefix_hi"]
    if n == 1:
        return [hi]
    step = next(s for s in (7, 5, 3, 1) if math.gcd(s, n) == 1)
    return [lo + (hi - lo) * ((b * step + 2) % n) // (n - 1) for b in range(n)]


def _torch_dtype(case):
    return {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}[case["dtype"]]


def prepare(case, seed):
    s = SHAPES[case["shape"]]
    d, hd, ffn, vocab, layers, batch = s["d"], s["head_dim"], s["ffn"], s["vocab"], case["layers"], case["batch"]
    kvd, td = s["kv_heads"] * hd, _torch_dtype(case)
    T, topk = TREE_T[case["tree"]], TREE_TOPK[case["tree"]]
    gen = torch.Generator(DEV).manual_seed(seed)
    cpu = torch.Generator().manual_seed(seed)

    def normal(*shape, std=1.0, dtype=td):
        return torch.empty(*shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=gen)

    gain = lambda: (1.0 + normal(d, std=0.3, dtype=torch.float32)).to(td)  # noqa: E731
    model = P.DeviceModel(d=d, n_heads=s["n_heads"], head_dim=hd, ffn=ffn, vocab=vocab, n_layers=layers, dtype=case["dtype"],
                          tree=case["tree"], n_kv_heads=s["kv_heads"], device=DEV, ffn_f16=case["ffn_f16"])
    st = dict(case=case, model=model)
    what, with_heads = case["what"], case["what"] == "heads" or case["heads"]
    if what != "heads":
        out_std = 0.02 / math.sqrt(2.0 * layers)
        for _ in range(layers):
            model.add_layer(normal(d, d, std=0.02), normal(kvd, d, std=0.02), normal(kvd, d, std=0.02), normal(d, d, std=out_std),
                            normal(ffn, d, std=0.02), normal(ffn, d, std=0.02), normal(d, ffn, std=out_std), gain(), gain())
    lm = normal(vocab, d, std=0.02) if what != "layer" else None

    if what == "step":
        # Tree tokens: all distinct.  Node n's own successor is a token of its own, except along one path of the tree down to
        # some depth, where the successor of a node is its child there: the continuation that the step accepts.
        info = P.medusa_tree_tables(model.tree)
        ids = torch.randperm(vocab, generator=cpu)[: min(vocab, 2 * batch * T)].to(DEV)
        tokens, succ = ids[: batch * T].view(batch, T), ids[batch * T:].view(batch, T).clone()
        if not case["heads"]:
            for b in range(batch):
                path = info["retrieve"][int(torch.randint(len(info["retrieve"]), (1,), generator=cpu))]
                path = [int(n) for n in path if n >= 0]
                depth = int(torch.randint(len(path), (1,), generator=cpu))
                for parent, child in zip(path[:depth], path[1: depth + 1]):
                    succ[b, parent] = tokens[b, child]
        embed = normal(vocab, d)
        if not case["heads"]:
            flat = succ.reshape(-1)
            lm[flat] = (lm[flat].float() + 0.01 * embed[tokens.reshape(-1)].float()).to(td)
        model.set_embed(embed)
        model.set_final_gain(gain())
        st["tokens"] = tokens.to(torch.int32).contiguous()
        del embed
    if what != "layer":
        model.set_lm_head(lm)
        del lm

    if with_heads:
        hidden = normal(batch, 1, d)
        st["hidden"] = hidden
        st["root"] = torch.randint(vocab, (batch,), generator=cpu).to(torch.int32).to(DEV)
        for k in topk:
            hl = normal(vocab, d, std=0.02)
            if what == "heads":  # the k candidates stand out from the vocabulary, one clearly above the next
                for b in range(batch):
                    rows = torch.randperm(vocab, generator=cpu)[:k].to(DEV)
                    lift = 0.006 - 0.0002 * torch.arange(k, device=DEV, dtype=torch.float32)
                    h = hidden[b, 0].float()
                    hl[rows] = (lift[:, None] * h[None, :]).to(td)
            model.add_medusa_head(normal(d, d, std=0.02), None, hl)
            del hl
    model.finalize()

    if what == "heads":
        st["buf"] = P.StepBuffers(model, batch, 0, want_head_logits=True)
        return st

    lengths = _prefixes(case)
    st["max_prefix"] = max(lengths) + 64
    kv = P.DeviceKV(model, batch, st["max_prefix"] + T, quant="fp8e4m3" if case["kv8"] else "")
    for l in range(layers):
        for b, n in enumerate(lengths):
            kv.write(l, b, 0, normal(s["kv_heads"], n, hd), normal(s["kv_heads"], n, hd))
    st["kv"] = kv
    st["lengths"] = torch.tensor(lengths, dtype=torch.int32, device=DEV)
    st["seq_len"] = st["lengths"].clone()
    if what == "layer":
        st["x0"] = normal(batch * T, d, dtype=torch.float32)
        st["x"] = torch.empty_like(st["x0"])
        st["ws"] = model.workspace(batch, st["max_prefix"])
    else:
        st["buf"] = P.StepBuffers(model, batch, st["max_prefix"], want_logits=case["logits"], want_head_logits=case["heads"])
        if not case["heads"]:
            st["buf"].tree_tokens.copy_(st["tokens"])
    return st


def _cache(st):
    """The cache's own buffers: numbers where rows are stored plainly, bytes where they are 8-bit codes."""
    kv, td = st["kv"], st["model"].tdtype
    return (kv.k, kv.v) if st["case"]["kv8"] else (kv.k.view(td), kv.v.view(td))


def run(st):
    case, model = st["case"], st["model"]
    if case["what"] == "heads":
        b = st["buf"]
        P.medusa_heads(model.desc, model.weights, st["hidden"], None, st["root"], case["batch"], 1, b.cand_flat, b.tree_tokens,
                       b.head_logits, b.ws)
        return dict(candidates=b.cand_flat, tree_tokens=b.tree_tokens, logits=b.head_logits[:, 1:])
    kv = st["kv"]
    if case["what"] == "layer":
        st["x"].copy_(st["x0"])
        P.tree_verify_layer(model.desc, model.layer(0), 0, st["x"], kv.desc, st["lengths"], case["batch"], st["max_prefix"], st["ws"])
        k, v = _cache(st)
        return dict(x=st["x"], k=k, v=v)
    b = st["buf"]
    st["seq_len"].copy_(st["lengths"])  # the lengths this step starts from, as a scheduler hands them over
    P.run_step(model, kv, b, st.get("hidden"), None, st.get("root"), st["seq_len"], with_heads=case["heads"])
    k, v = _cache(st)
    out = dict(node_argmax=b.node_argmax, hidden=b.hidden, accept_len=b.accept_len, best_path=b.best_path, acc_nodes=b.acc_nodes,
               acc_tokens=b.acc_tokens, next_root=b.next_root, last_node=b.last_node, src_slots=b.kv_src_slots,
               seq_len=st["seq_len"], k=k, v=v)
    if case["logits"]:
        out["logits"] = b.logits
    if case["heads"]:
        out.update(candidates=b.cand_flat, tree_tokens=b.tree_tokens, head_logits=b.head_logits[:, 1:])
    return out


def work(case):
    s = SHAPES[case["shape"]]
    d, hd, ffn, vocab, batch = s["d"], s["head_dim"], s["ffn"], s["vocab"], case["batch"]
    kvd, es, layers = s["kv_heads"] * hd, 4 if case["dtype"] == "fp32" else 2, case["layers"]
    T, topk = TREE_T[case["tree"]], TREE_TOPK[case["tree"]]
    rows = batch * T
    nbytes = flops = 0
    if case["what"] == "heads" or case["heads"]:
        n = len(topk) * (d * d + d * vocab)
        nbytes += n * es + batch * (d * es + len(topk) * vocab * 4)
        flops += 2 * batch * n
    if case["what"] == "heads":
        return {"bytes": nbytes, "flops": flops}
    layer = d * (d + 2 * kvd) + d * d + 3 * d * ffn
    row = 132 / 128 * hd if case["kv8"] else hd * es  # bytes of one cache row of one head
    lengths = _prefixes(case)
    nbytes += layers * (layer * es + sum(lengths) * 2 * s["kv_heads"] * row + rows * 2 * s["kv_heads"] * row)
    flops += layers * (2 * rows * layer + sum(4 * T * (n + T) * d for n in lengths))
    if case["what"] == "layer":
        return {"bytes": nbytes + 2 * rows * d * 4, "flops": flops}
    nbytes += vocab * d * es + 2 * rows * d * es + (rows * vocab * 4 if case["logits"] else 0)
    flops += 2 * rows * d * vocab
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Two orders of summation (the same step with its attention in another kernel order) were measured apart by 6.2e-3 in the
    # 2-norm (bf16, 32 layers; largest single difference 4.7e-2 of the root mean square), 8e-4 and 6e-3 in fp16; fp32 is held
    # to the rounding of its sums.  About three to four times that is allowed.  Whole numbers are decided by margins far above
    # it; bytes of 8-bit cache rows may land on the neighbouring code (measured: 0.09 % of them).
    rel, most = {"fp32": (1e-5, 1e-4), "bf16": (2e-2, 0.2), "fp16": (3e-3, 0.03)}[case["dtype"]]
    return {"rel": rel, "max": most, "differ": 0.004 if case["kv8"] else 0.0}
