"""What a row without an edge to a node must not see of that node: scores above any finite mask, infinities and NaNs, and
softmax scales so small that a masked score would come back into range."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_04070_amd import binding as bpt
from paper_1911_04070_amd.workloads import Workload, make_inputs
from test_gpu_parity import host, say, to_dev, tol_for

pytestmark = pytest.mark.gpu

# bias tables of the bf16 token tiles: staged, as a ring, out of memory (by pairs and, with lengths, at once)
BF16 = [(256, 4, False), (512, 8, True), (512, 24, False), (512, 80, False)]


@pytest.mark.parametrize("shorter", [False, True])
@pytest.mark.parametrize("n,k,causal", BF16)
def test_bf16_small_scale(n, k, causal, shorter):
    # scale times any mask that is a finite number is no mask: every row has to be the mean of its neighbours' values.
    # (dQ, dK and d_rel carry the factor scale: nothing but zeros here)
    say("small scale", n, k, causal, shorter)
    scale = 1e-30
    lengths = [n - n // 3, n] if shorter else [n, n]
    x = make_inputs(Workload("small_scale", 15, n, k, causal, 2, 2, 64, "bf16", True))
    g = bpt.bpt_build_graph(n, k, causal)
    kw = dict(scale=scale, seq_len=torch.tensor(lengths, dtype=torch.int32, device="cuda") if shorter else None)
    d = {key: to_dev(v, "bf16") for key, v in x.items()}
    out, lse = bpt.bpt_attn_fwd(g, d["Q"], d["K"], d["V"], d["Rel"], **kw)
    _, _, dV, _ = bpt.bpt_attn_bwd(g, d["Q"], d["K"], d["V"], d["Rel"], lse, d["dO"], **kw)
    o, l, _ = oracle.attn_fwd_lengths(n, k, causal, lengths, x["Q"], x["K"], x["V"], x["Rel"], scale)
    refs = oracle.attn_bwd_lengths(n, k, causal, lengths, x["Q"], x["K"], x["V"], x["Rel"], x["dO"], scale)
    for name, got, ref in (("out", out, o), ("lse", lse, l), ("dV", dV, refs[2])):
        assert np.abs(host(got) - ref).max() <= tol_for("bf16", ref, scaled=True), name
    g.destroy()


def reads_of(g, nodes):
    """rows that have an edge to one of the nodes"""
    row_ptr, col, _ = g.csr_to_host()
    rows = np.repeat(np.arange(len(row_ptr) - 1), np.diff(row_ptr))
    hit = np.zeros(len(row_ptr) - 1, bool)
    hit[rows[np.isin(col, nodes)]] = True
    return hit


def keys_of(g, rows):
    """nodes that one of the rows (a mask) has an edge to"""
    row_ptr, col, _ = g.csr_to_host()
    row = np.repeat(np.arange(len(row_ptr) - 1), np.diff(row_ptr))
    hit = np.zeros(len(row_ptr) - 1, bool)
    hit[col[rows[row]]] = True
    return hit


def bad_nodes(n):
    """tokens at both ends and in the middle of a tile, spans of a low and a high level"""
    return np.array([0, n // 2 + 5, n - 1, n + n // 4 + 3, 2 * n - 3])


NAN, INF = float("nan"), float("inf")


@pytest.mark.parametrize("value", [NAN, INF, 1e37])
@pytest.mark.parametrize("kind", ["full", "lengths", "dropout", "packed"])
@pytest.mark.parametrize("n,k,causal", BF16)
def test_bf16_keys_of_other_rows(n, k, causal, kind, value):
    # forward, bf16: a K row reaches the rows with an edge to it; the others keep every bit
    say("bf16", n, k, causal, kind, value)
    w = Workload("masked", 15, n, k, causal, 2, 2, 64, "bf16", False)
    x = make_inputs(w)
    g = bpt.bpt_build_graph(n, k, causal)
    bad = bad_nodes(n)
    kw = {}
    if kind == "lengths":
        kw["seq_len"] = torch.tensor([n, n - n // 4], dtype=torch.int32, device="cuda")
        bad = bad[:2]      # (nodes that a sequence does not keep have to hold finite values)
    if kind == "dropout":
        kw["dropout"] = (0.2, 3)
    Q, K, V, R = (to_dev(x[key], "bf16") for key in ("Q", "K", "V", "Rel"))
    if kind == "packed":   # one sequence of n tokens: the rows of the tree itself, through the packed kernels
        pg = bpt.bpt_build_batch_graph(n, k, causal, [n])
        assert pg.num_nodes == g.num_nodes
        Q, K, V = (t[:1].contiguous() for t in (Q, K, V))
    graph = pg if kind == "packed" else g
    out0, lse0 = bpt.bpt_attn_fwd(graph, Q, K, V, R, **kw)
    K[:, :, torch.from_numpy(bad).cuda()] = value
    out, lse = bpt.bpt_attn_fwd(graph, Q, K, V, R, **kw)
    other = torch.from_numpy(~reads_of(g, bad)).cuda()
    assert int(other.sum()) > 0
    assert torch.equal(out[:, :, other], out0[:, :, other])
    assert torch.equal(lse[:, :, other], lse0[:, :, other])
    graph.destroy()


# sizes of the fp32 tiles: fewer chunks than wavefronts, rows of all kinds of span segments, ids on either side of the
# query side's variants (up to 96, 192, 384 and gather), key tiles cut into several tasks
F32 = [(32, 3, True), (256, 8, False), (512, 7, True), (1024, 25, False), (512, 59, False), (4096, 2, False)]


F32_KINDS = [("full", c, v) for c in F32 for v in (NAN, -INF)] + [(kind, c, -INF) for kind in ("lengths", "dropout", "packed") for c in F32[:3]]


@pytest.mark.parametrize("what", ["K", "V", "Q", "dO"])
@pytest.mark.parametrize("kind,graph,value", F32_KINDS)
def test_f32_reaches_only_neighbours(kind, graph, value, what):
    # the tiles (full) and the gather kernels (the rest)
    n, k, causal = graph
    say("f32", n, k, causal, kind, value, what)
    B, H = 1, 2
    w = Workload("masked", 15, n, k, causal, B, H, 64, "f32", True)
    x = make_inputs(w)
    g = bpt.bpt_build_graph(n, k, causal)
    bad = bad_nodes(n)
    kw, okw = {}, {}
    if kind == "lengths":
        kw["seq_len"] = torch.tensor([n - n // 4], dtype=torch.int32, device="cuda")
        bad = bad[:2]      # (nodes that a sequence does not keep have to hold finite values)
    if kind == "dropout":
        kw["dropout"], okw = (0.2, 3), dict(dropout=0.2, seed=3)
    lengths = [n - n // 4 if kind == "lengths" else n] * B
    o, l, _ = oracle.attn_fwd_lengths(n, k, causal, lengths, x["Q"], x["K"], x["V"], x["Rel"], w.scale, **okw)
    refs = oracle.attn_bwd_lengths(n, k, causal, lengths, x["Q"], x["K"], x["V"], x["Rel"], x["dO"], w.scale, **okw)
    d = {key: to_dev(x[key], "f32") for key in ("Q", "K", "V", "dO", "Rel")}
    d[what][:, :, torch.from_numpy(bad).cuda()] = value
    graph = bpt.bpt_build_batch_graph(n, k, causal, [n]) if kind == "packed" else g
    out, lse = bpt.bpt_attn_fwd(graph, d["Q"], d["K"], d["V"], d["Rel"], scale=w.scale, **kw)
    grads = bpt.bpt_attn_bwd(graph, d["Q"], d["K"], d["V"], d["Rel"], lse, d["dO"], scale=w.scale, **kw)
    torch.cuda.synchronize()
    own = np.zeros(g.num_nodes, bool)
    own[bad] = True
    rows = reads_of(g, bad) if what in ("K", "V") else own          # rows with a score or a value that is not finite
    forward = rows if what != "dO" else np.zeros_like(rows)
    touched = dict(out=forward, lse=forward if what in ("K", "Q") else np.zeros_like(rows), dQ=rows, dK=keys_of(g, rows) | own,
                   dV=keys_of(g, rows) | own)
    for name, got, ref in zip(("out", "lse", "dQ", "dK", "dV"), (out, lse) + tuple(grads), (o, l) + tuple(refs)):
        a, keep = host(got), ~touched[name]
        assert keep.any() or n <= 32, name
        assert np.isfinite(a[:, :, keep]).all(), name
        if keep.any():
            assert np.abs(a[:, :, keep] - ref[:, :, keep]).max() <= tol_for("f32", ref[:, :, keep], scaled=True), name
    if what == "V" and kind == "full":   # and it does reach the rows it belongs to
        assert not np.isfinite(host(out)[:, :, rows]).all(-1).any()
    graph.destroy()
