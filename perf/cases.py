"""The work users have this library do, as cases that can be timed.

A case names a path ("kind") and its sizes:

  attention  bpt_attn_fwd [+ bpt_attn_bwd] into buffers the program keeps, as bench.py's step and the layer call them
  autograd   graph_attention and its backward: the torch entry point, on a padded batch of sentences
  packed     attention over one graph for a batch of sequences of different lengths, gradients in bf16
  layer      one training step of the graph layer (forward + backward, all parameter gradients)
  stack      the update of the graph over several layers: inference on a batch of sequences, or a training step on a
             packed batch whose graph is built in the pass, as a loop over batches of sentences does

`listed()` spans the sizes of paper_1911_04070_amd/workloads.py and bench.py; `draw()` gives other sizes of the same
ranges.  Values: Q, K, V, dO and states are N(0, 1), relative-position tables N(0, 0.02^2), parameters as a fresh
layer has them -- the distributions of the tests and the benchmark.
"""
import math

import torch

from paper_1911_04070_amd import binding as bpt

HEAD = 64
FFN_FACTOR = 4


def listed():
    return [
        # one short sequence in fp32, forward only: nothing but launches and latency
        dict(name="tiny_f32", kind="attention", n=512, k=4, causal=False, B=1, H=1, dtype="f32", backward=False, dropout=0.0),
        # fp32 training of a small model: the precision of gradient checks and of models that do not train in bf16
        dict(name="train_f32", kind="attention", n=2048, k=8, causal=True, B=2, H=8, dtype="f32", backward=True, dropout=0.0),
        # a batch of 32 sentences of different lengths padded to 512, through torch's autograd
        dict(name="sentences", kind="autograd", n=512, k=4, causal=False, B=32, H=8),
        # the classification shape, every sequence full
        dict(name="cls", kind="attention", n=512, k=4, causal=False, B=32, H=8, dtype="bf16", backward=True, dropout=0.0),
        # long-context language modelling, training and inference
        dict(name="lm", kind="attention", n=8192, k=8, causal=True, B=4, H=8, dtype="bf16", backward=True, dropout=0.0),
        dict(name="lm_infer", kind="attention", n=8192, k=8, causal=True, B=4, H=8, dtype="bf16", backward=False, dropout=0.0),
        # extreme length
        dict(name="xl", kind="attention", n=65536, k=4, causal=True, B=1, H=8, dtype="bf16", backward=True, dropout=0.0),
        # a denser bidirectional graph, with dropout on the attention weights
        dict(name="dense_dropout", kind="attention", n=4096, k=16, causal=False, B=8, H=8, dtype="bf16", backward=True, dropout=0.1),
        # the density of character-level language models
        dict(name="charlm", kind="attention", n=8192, k=64, causal=True, B=4, H=8, dtype="bf16", backward=True, dropout=0.0),
        # eight documents of very different lengths in one packed graph
        dict(name="packed_lm", kind="packed", n=8192, k=8, causal=True, B=8, H=8),
        # a training step of two layers on packed sentences, the graph of the batch built in the step
        dict(name="stack_train", kind="stack", n=512, k=4, causal=False, B=32, H=8, layers=2, packed=True, backward=True),
        # one layer on the language-model shape, training
        dict(name="layer_lm", kind="layer", n=8192, k=8, causal=True, B=4, H=8),
    ]


def draw(rng):
    def size(lo, hi):        # whole number, its logarithm spread evenly, odd ones among them
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def tokens(lo, hi):      # the trees are over powers of two
        return 1 << rng.randint(lo.bit_length() - 1, hi.bit_length() - 1)

    def fit(n, most):        # batch and heads with B * H * n <= most
        H = rng.choice([1, 2, 3, 4, 5, 6, 8, 8, 8, 12, 16])
        while H > 1 and H * n > most:
            H //= 2
        return size(1, max(1, min(32, most // (H * n)))), H

    what = rng.choice(["f32", "f32", "sentences", "train", "train", "train", "infer", "packed", "stack_train", "stack_infer", "layer"])
    causal = rng.random() < 0.5
    if what == "f32":
        n = tokens(64, 4096)
        B, H = fit(n, 1 << 15)
        return dict(kind="attention", n=n, k=size(1, 16), causal=causal, B=B, H=H, dtype="f32", backward=rng.random() < 0.6, dropout=0.0)
    if what == "sentences":
        return dict(kind="autograd", n=tokens(64, 1024), k=size(1, 8), causal=causal, B=rng.randint(3, 32), H=rng.randint(1, 8))
    if what in ("train", "infer"):
        n = tokens(256, 65536)
        B, H = fit(n, 1 << 18 if n < 65536 else 1 << 19)
        k = size(1, 64 if causal and n <= 8192 else 32 if n <= 4096 else 12)
        return dict(kind="attention", n=n, k=k, causal=causal, B=B, H=H, dtype="bf16", backward=what == "train",
                    dropout=rng.choice([0.0, 0.0, 0.1, 0.2]) if what == "train" else 0.0)
    if what == "packed":
        n = tokens(512, 8192)
        B, H = fit(n, 1 << 18)
        return dict(kind="packed", n=n, k=size(2, 16), causal=causal, B=max(2, B), H=H)
    if what == "stack_train":
        n = tokens(64, 1024)
        return dict(kind="stack", n=n, k=size(2, 8), causal=causal, B=rng.randint(3, max(4, min(32, (1 << 14) // n))), H=rng.choice([2, 4, 6, 8]),
                    layers=rng.randint(1, 3), packed=True, backward=True)
    if what == "stack_infer":   # 8192 tokens per batch, the sequence length varied
        n = tokens(256, 8192)
        return dict(kind="stack", n=n, k=size(1, 16), causal=causal, B=8192 // n, H=rng.choice([4, 8]), layers=rng.randint(2, 6), packed=False,
                    backward=False)
    n = tokens(256, 8192)
    return dict(kind="layer", n=n, k=size(2, 16), causal=causal, B=rng.randint(1, max(1, (1 << 15) // n)), H=rng.choice([2, 4, 6, 8]))


# ---- inputs ---------------------------------------------------------------------------------------------
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(gen, shape, dtype, std=1.0):
    x = torch.randn(shape, device="cuda", generator=gen, dtype=torch.float32)
    return (x if std == 1.0 else x.mul_(std)).to(dtype)


def _lengths(case, seed):
    """Token counts of the B sequences: the B quantiles of a log-normal with median 0.4 n and sigma 0.6, clipped to
    [8, n], in an order of the seed's."""
    B, n = case["B"], case["n"]
    q = (torch.arange(B, dtype=torch.float64) + 0.5) / B
    x = (0.4 * n * torch.exp(0.6 * math.sqrt(2.0) * torch.erfinv(2 * q - 1))).round().clamp(8, n).to(torch.int32)
    return x[torch.randperm(B, generator=torch.Generator().manual_seed(seed))]


def _table(gen, g, dtype):
    return _normal(gen, (g.num_levels, g.rel_width, HEAD), dtype, 0.02)


def _parameters(gen, d, d_ff):
    p = {w: _normal(gen, (d, d), torch.bfloat16, d ** -0.5) for w in ("Wq", "Wk", "Wv", "Wo")}
    p["W1"] = _normal(gen, (d, d_ff), torch.bfloat16, d ** -0.5)
    p["W2"] = _normal(gen, (d_ff, d), torch.bfloat16, d_ff ** -0.5)
    p["b1"] = _normal(gen, (d_ff,), torch.float32, 0.1)
    p["b2"] = _normal(gen, (d,), torch.float32, 0.1)
    for gain, shift in (("g1", "beta1"), ("g2", "beta2")):
        p[gain] = 1.0 + _normal(gen, (d,), torch.float32, 0.1)
        p[shift] = _normal(gen, (d,), torch.float32, 0.1)
    return p


def _bytes(count):
    return torch.empty(max(count, 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    return {"attention": _prepare_attention, "autograd": _prepare_autograd, "packed": _prepare_packed, "layer": _prepare_layer,
            "stack": _prepare_stack}[case["kind"]](case, seed)


def run(state):
    return state["run"](state)


def _prepare_attention(case, seed):
    gen = _generator(seed)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    g = bpt.bpt_build_graph(case["n"], case["k"], case["causal"])
    shape = (case["B"], case["H"], g.num_nodes, HEAD)
    s = dict(run=_run_attention, g=g, rel=_table(gen, g, dt), dropout=(case["dropout"], seed & 0xFFFFFFFF) if case["dropout"] else None)
    for name in ("Q", "K", "V"):
        s[name] = _normal(gen, shape, dt)
    s["out"], s["lse"] = torch.empty_like(s["Q"]), torch.empty(shape[:3], dtype=torch.float32, device="cuda")
    fws, bws = bpt.workspace_bytes(g, s["Q"])
    s["fws"] = _bytes(fws)
    s["dO"] = None
    if case["backward"]:
        s["dO"] = _normal(gen, shape, dt)
        s["bws"] = _bytes(bws)
        s["grads"] = tuple(torch.empty(shape, dtype=torch.float32, device="cuda") for _ in range(3)) + (
            torch.empty(s["rel"].shape, dtype=torch.float32, device="cuda"),)
    return s


def _run_attention(s):
    bpt.bpt_attn_fwd(s["g"], s["Q"], s["K"], s["V"], s["rel"], out=s["out"], lse=s["lse"], workspace=s["fws"], dropout=s["dropout"])
    if s["dO"] is None:
        return s["out"], s["lse"]
    bpt.bpt_attn_bwd(s["g"], s["Q"], s["K"], s["V"], s["rel"], s["lse"], s["dO"], grads=s["grads"], workspace=s["bws"], dropout=s["dropout"])
    return (s["out"], s["lse"]) + s["grads"]


def _prepare_autograd(case, seed):
    gen = _generator(seed)
    g = bpt.bpt_build_graph(case["n"], case["k"], case["causal"])
    shape = (case["B"], case["H"], g.num_nodes, HEAD)
    s = dict(run=_run_autograd, g=g, lengths=_lengths(case, seed).cuda(), dO=None)
    s["leaves"] = [_normal(gen, shape, torch.bfloat16).requires_grad_() for _ in range(3)] + [_table(gen, g, torch.bfloat16).requires_grad_()]
    s["dO"] = _normal(gen, shape, torch.bfloat16)
    return s


def _run_autograd(s):
    out = bpt.graph_attention(s["g"], *s["leaves"], seq_len=s["lengths"])
    return (out.detach(),) + torch.autograd.grad(out, s["leaves"], s["dO"])


def _prepare_packed(case, seed):
    gen = _generator(seed)
    g = bpt.bpt_build_batch_graph(case["n"], case["k"], case["causal"], _lengths(case, seed).numpy())
    shape = (1, case["H"], g.num_nodes, HEAD)
    s = dict(run=_run_packed, g=g, rel=_table(gen, g, torch.bfloat16))
    for name in ("Q", "K", "V", "dO"):
        s[name] = _normal(gen, shape, torch.bfloat16)
    s["out"], s["lse"] = torch.empty_like(s["Q"]), torch.empty(shape[:3], dtype=torch.float32, device="cuda")
    s["grads"] = tuple(torch.empty_like(s["Q"]) for _ in range(3)) + (torch.empty(s["rel"].shape, dtype=torch.float32, device="cuda"),)
    fws, bws = bpt.workspace_bytes(g, s["Q"])
    s["fws"], s["bws"] = _bytes(fws), _bytes(bws)
    return s


def _run_packed(s):
    bpt.bpt_attn_fwd(s["g"], s["Q"], s["K"], s["V"], s["rel"], out=s["out"], lse=s["lse"], workspace=s["fws"])
    bpt.bpt_attn_bwd(s["g"], s["Q"], s["K"], s["V"], s["rel"], s["lse"], s["dO"], grads=s["grads"], workspace=s["bws"])
    return (s["out"], s["lse"]) + s["grads"]


def _prepare_layer(case, seed):
    gen = _generator(seed)
    g = bpt.bpt_build_graph(case["n"], case["k"], case["causal"])
    d = case["H"] * HEAD
    shape = (case["B"], g.num_nodes, d)
    fws, bws = bpt.layer_workspace_bytes(g, case["B"], case["H"], FFN_FACTOR * d)
    s = dict(run=_run_layer, g=g, H=case["H"], rel=_table(gen, g, torch.bfloat16), p=_parameters(gen, d, FFN_FACTOR * d),
             X=_normal(gen, shape, torch.bfloat16), dY=_normal(gen, shape, torch.bfloat16), fws=_bytes(fws), bws=_bytes(bws))
    s["Y"] = torch.empty_like(s["X"])
    return s


def _run_layer(s):
    bpt.bpt_layer_fwd(s["g"], s["X"], s["rel"], s["p"], s["H"], out=s["Y"], workspace=s["fws"])
    return (s["Y"],) + tuple(bpt.bpt_layer_bwd(s["g"], s["X"], s["rel"], s["p"], s["H"], s["fws"], s["dY"], workspace=s["bws"]))


def _prepare_stack(case, seed):
    gen = _generator(seed)
    tree = bpt.bpt_build_graph(case["n"], case["k"], case["causal"])
    d = case["H"] * HEAD
    s = dict(run=_run_stack_training if case["backward"] else _run_stack_inference, tree=tree, H=case["H"], d_ff=FFN_FACTOR * d,
             rels=[_table(gen, tree, torch.bfloat16) for _ in range(case["layers"])],
             p=[_parameters(gen, d, FFN_FACTOR * d) for _ in range(case["layers"])])
    if case["packed"]:
        s["lengths"] = _lengths(case, seed).numpy()
        s["E"] = _normal(gen, (1, int(s["lengths"].sum()), d), torch.bfloat16)
        s["d_root"] = _normal(gen, (case["B"], d), torch.bfloat16)
    else:
        s["E"] = _normal(gen, (case["B"], case["n"], d), torch.bfloat16)
        s["fws"] = _bytes(bpt.stack_workspace_bytes(tree, case["B"], case["H"], FFN_FACTOR * d, case["layers"])[0])
    return s


def _run_stack_training(s):
    g = bpt.bpt_build_batch_graph_on(s["tree"], s["lengths"])
    fws, bws = bpt.stack_workspace_bytes(g, 1, s["H"], s["d_ff"], len(s["p"]))
    fws, bws = _bytes(fws), _bytes(bws)
    root, _ = bpt.bpt_stack_fwd(g, s["E"], s["rels"], s["p"], s["H"], want_tokens=False, workspace=fws)
    dE, d_rels, grads = bpt.bpt_stack_bwd(g, s["E"], s["rels"], s["p"], s["H"], fws, s["d_root"], None, workspace=bws)
    return root, dE, d_rels, grads


def _run_stack_inference(s):
    root, tokens = bpt.bpt_stack_fwd(s["tree"], s["E"], s["rels"], s["p"], s["H"], workspace=s["fws"])
    return root, tokens


# ---- what a pass cannot do without ----------------------------------------------------------------------
def _rows_and_edges(case):
    """(node rows, edges) of the case's batch, one head: the nodes that exist and the edges between them."""
    n, k, causal = case["n"], case["k"], case["causal"]
    if case["kind"] in ("autograd", "packed") or case.get("packed"):
        lengths = [int(x) for x in _lengths(case, 0)]
        rows = sum((x + (1 << level) - 1) >> level for x in lengths for level in range(n.bit_length()))
        return rows, sum(bpt.bpt_count_edges(n, k, causal, x) for x in lengths)
    return case["B"] * (2 * n - 1), case["B"] * bpt.bpt_count_edges(n, k, causal, n)


def _attention_work(rows, edges, H, width, backward, grad_width):
    """Each of Q, K, V (and dO) read once, out and lse (and dQ, dK, dV) written once; per edge and head the products
    q.k, q.r and p v forward, those of dP, dQ (keys and table), dK, dV and d_rel backward (scores are not formed again)."""
    size = rows * H * (HEAD * 4 * width + 4)
    flops = edges * H * 3 * 2 * HEAD
    if backward:
        size += rows * H * HEAD * (width + 3 * grad_width)
        flops += edges * H * 6 * 2 * HEAD
    return size, flops


def work(case):
    rows, edges = _rows_and_edges(case)
    H, kind = case["H"], case["kind"]
    if kind in ("attention", "autograd", "packed"):
        width = 4 if case.get("dtype") == "f32" else 2
        size, flops = _attention_work(rows, edges, H, width, case.get("backward", True), 4 if kind == "attention" else 2)
        return {"bytes": size, "flops": flops}
    d = H * HEAD
    d_ff = FFN_FACTOR * d
    layers, backward = case.get("layers", 1), case.get("backward", True)
    weights = 4 * d * d + 2 * d * d_ff
    _, attn = _attention_work(rows, edges, H, 2, backward, 2)
    flops = layers * (2 * rows * weights * (3 if backward else 1) + attn)
    states = rows * d * 2 if kind == "layer" else rows * d      # a stack reads and writes token rows: about half
    # (bytes: states in and out, weights and their fp32 gradients; in training the dense maps' gradients are products
    # of the states with what came after them, so the states are held, not counted again)
    size = states * (4 if backward else 2) + layers * weights * (2 + 4 if backward else 2)
    return {"bytes": size, "flops": flops}


def tolerance(case):
    """Four times the largest relative error seen: fp32 against the oracle in 64 bits 3.3e-7 (d_rel); bf16 `out` against
    it 1.8e-3 (its own rounding); layers and stacks between the two GEMM libraries they can run on 1e-2 and more (dW1:
    a hidden unit near zero that takes the other side of the ReLU changes its gradient by all of it)."""
    if case["kind"] == "attention" and case["dtype"] == "f32":
        return {"rel": 2e-6}
    if case["kind"] in ("layer", "stack"):
        return {"rel": 0.03 if case.get("backward", True) else 2.5e-2}
    return {"rel": 8e-3}
