"""GPU parity: the HIP library (through its C ABI) against the CPU oracle.

Graph arrays must be bit-identical.  Attention must agree within max-abs 1e-4
for fp32 tensors and 2e-2 for bf16 tensors with fp32 accumulation (the
tolerances the benchmark spec fixes), as absolute bounds on every output.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_04070_amd import binding as bpt
from paper_1911_04070_amd.workloads import WORKLOADS, Workload, make_inputs, shrink

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


def say(*a):
    print(*a, flush=True)


def tol_for(dtype, ref, scaled=False):
    """max-abs tolerance of the benchmark spec: 1e-4 for fp32 tensors, 2e-2 for bf16 tensors.  These are absolute bounds for
    the task's N(0, 1) inputs, whose results have entries up to about 4; `scaled` (inputs made larger on purpose)
    lets the bound grow with the largest entry of the expected tensor beyond that."""
    return TOL[dtype] * (max(1.0, float(np.abs(ref).max()) / 4.0) if scaled else 1.0)


def to_dev(x, dtype):
    t = torch.from_numpy(np.ascontiguousarray(x))
    if dtype == "bf16":
        t = t.to(torch.bfloat16)              # exact: values are already bf16-representable
    return t.cuda()


def host(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


GRAPHS = [(2, 1, False), (2, 1, True), (4, 1, False), (8, 3, True), (16, 2, False), (64, 64, False), (64, 100, True),
          (512, 4, False), (1024, 1, False), (2048, 100, True), (8192, 8, True), (65536, 4, True)] + \
         [(4096, k, False) for k in (2, 4, 8, 16, 32)] + [(262144, 2, False), (1048576, 1, True)]   # 25 M and 50 M edges


@pytest.mark.parametrize("n,k,causal", GRAPHS)
def test_graph_is_bit_exact(n, k, causal):
    say("graph", n, k, causal)
    ref = oracle.build_graph(n, k, causal)
    g = bpt.bpt_build_graph(n, k, causal)
    assert (g.num_nodes, g.num_edges, g.num_levels, g.rel_width) == (ref.num_nodes, ref.num_edges, ref.num_levels,
                                                                      ref.rel_width)
    row_ptr, col, rel = g.csr_to_host()
    assert np.array_equal(row_ptr, ref.row_ptr)
    assert np.array_equal(col, ref.col)
    assert np.array_equal(rel, ref.rel)
    t_ptr, t_src, t_eid = g.transposed_to_host()
    r_ptr, r_src, r_eid = oracle.transpose(ref)
    assert np.array_equal(t_ptr, r_ptr)
    assert np.array_equal(t_src, r_src)
    assert np.array_equal(t_eid, r_eid)
    # levels on which some token has contextual nodes
    lv = ref.rel[:ref.row_ptr[n]] // ref.rel_width
    assert g.ctx_levels == int(lv.max()) + 1
    g.destroy()


def test_graph_errors_on_device():
    import ctypes
    L = bpt.load_library()
    h = ctypes.c_void_p()
    # complete token graph at n = 65536 has n^2 > INT32_MAX edges
    assert L.bpt_build_graph(65536, 65536, 0, None, ctypes.byref(h)) == bpt.BPT_ERR_OVERFLOW
    assert h.value is None
    with pytest.raises(bpt.BptError):
        bpt.bpt_build_graph(48, 2, False)


def run_case(w: Workload, x=None, layout="bhnd", check_bwd=None, scaled=False):
    """Runs forward (+ backward) of a workload on the GPU and on the oracle and compares."""
    say("case", w)
    if x is None:
        x = make_inputs(w)
    ref_g = oracle.build_graph(w.n, w.k, w.causal)
    g = bpt.bpt_build_graph(w.n, w.k, w.causal)
    dev = {}
    for key in ("Q", "K", "V", "dO"):
        if key in x:
            t = to_dev(x[key], w.dtype)
            if layout == "bnhd":               # same logical tensor, node-major memory
                t = t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
            dev[key] = t
    rel_d = to_dev(x["Rel"], w.dtype)
    out_d, lse_d = bpt.bpt_attn_fwd(g, dev["Q"], dev["K"], dev["V"], rel_d, scale=w.scale)
    torch.cuda.synchronize()
    out_r, lse_r, _ = oracle.attn_fwd(ref_g, x["Q"], x["K"], x["V"], x["Rel"], w.scale)
    res = {}
    for name, got, ref in (("out", host(out_d), out_r), ("lse", host(lse_d), lse_r)):
        err = float(np.abs(got - ref).max())
        res[name] = err
        assert np.isfinite(got).all(), name
        assert err <= tol_for(w.dtype, ref, scaled), (name, err)
    do_bwd = w.backward if check_bwd is None else check_bwd
    if do_bwd:
        grads = bpt.bpt_attn_bwd(g, dev["Q"], dev["K"], dev["V"], rel_d, lse_d, dev["dO"], scale=w.scale)
        torch.cuda.synchronize()
        refs = oracle.attn_bwd(ref_g, x["Q"], x["K"], x["V"], x["Rel"], x["dO"], w.scale)
        for name, got_t, ref in zip(("dQ", "dK", "dV", "d_rel"), grads, refs[:4]):
            got = host(got_t)
            err = float(np.abs(got - ref).max())
            res[name] = err
            res[name + "_max"] = float(np.abs(ref).max())
            assert np.isfinite(got).all(), name
            assert err <= tol_for(w.dtype, ref, scaled), (name, err, float(np.abs(ref).max()))
        # r_anc never changes the output (it shifts a whole span row): its gradient is zero
        anc = host(grads[3])[1:, w.k + 1]
        assert np.abs(anc).max() <= TOL[w.dtype]
    say("   max-abs errors", {k: float("%.3g" % v) for k, v in res.items()})
    g.destroy()
    return res


def test_forward_tiny_fp32():
    # configuration 1: n=512, k=4, bidirectional, one head of 64, fp32, forward only
    run_case(WORKLOADS["tiny"])


SMALL = [
    ("f32", 2, 1, False, 1, 1), ("f32", 4, 1, True, 2, 1), ("f32", 8, 3, False, 1, 3), ("f32", 16, 2, False, 2, 2),
    ("f32", 64, 100, False, 1, 2), ("f32", 256, 3, True, 2, 3), ("f32", 2048, 5, False, 1, 2),
    ("bf16", 2, 1, True, 1, 1), ("bf16", 32, 2, False, 3, 2), ("bf16", 128, 200, True, 1, 2),
    ("bf16", 1024, 7, False, 2, 2), ("bf16", 4096, 3, True, 1, 3),
    # sizes around the switches of the tile kernels: no tiles (n < 16), token tiles without span
    # blocks (n = 16), span blocks without / with one / with several ancestor levels (n = 32, 64, 512),
    # one token tile per wavefront group left over (n = 16 * 5 is not a power of two: n = 256 with 5 (b, h))
    ("bf16", 8, 2, False, 2, 1), ("bf16", 16, 1, False, 1, 3), ("bf16", 16, 30, True, 2, 1),
    ("bf16", 32, 1, True, 1, 1), ("bf16", 64, 2, False, 1, 5), ("bf16", 64, 1, True, 5, 1),
    ("bf16", 256, 4, True, 1, 5), ("bf16", 512, 1, False, 1, 1), ("bf16", 2048, 16, False, 1, 1),
]


@pytest.mark.parametrize("dtype,n,k,causal,B,H", SMALL)
def test_forward_backward_small(dtype, n, k, causal, B, H):
    w = Workload("small", 7, n, k, causal, B, H, 64, dtype, True)
    run_case(w)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_strided_layout(dtype):
    # [B,N,H,D] memory (all heads of a node adjacent) through the stride arguments
    w = Workload("strided", 8, 512, 4, False, 2, 4, 64, dtype, True)
    run_case(w, layout="bnhd")


def test_rows_cut_into_several_segments():
    # n=4096, k=40: token rows of > 512 edges, span rows up to 4096, key nodes with
    # thousands of queries: every merge path runs
    w = Workload("segments", 9, 4096, 40, False, 1, 2, 64, "bf16", True)
    run_case(w)
    w = Workload("segments32", 9, 2048, 12, True, 1, 1, 64, "f32", True)
    run_case(w)


@pytest.mark.parametrize("n,k,causal", [(4096, 64, True), (1024, 72, False), (2048, 50, False)])
def test_large_density_on_key_tiles(n, k, causal):
    # the paper's character-level density k = 64 (Sec. 4.2) and the largest the key tiles take:
    # 7..10 blocks of 16 relative-position ids per level
    run_case(Workload("dense_k", 11, n, k, causal, 1, 2, 64, "bf16", True))


FULL = ["cls", "lm", "xl", "ksweep2", "ksweep4", "ksweep8", "ksweep16", "ksweep32", "charlm"]


# key tiles that meet 64, 80, 160 and (gather kernels) 176 ids: the last size with all table operands in registers,
# the first and last with the ones of the pair at hand; bidirectional tiles have pairs whose edges lie on both sides
# and on ancestors, so that two blocks of ids want the same registers
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("n,k", [(512, 26), (512, 27), (128, 40), (1024, 73), (1024, 74)])
def test_key_tiles_of_many_ids(n, k, causal):
    w = Workload("keys%d" % k, 9, n, k, causal, 1, 2, 64, "bf16", True)
    x = make_inputs(w)
    x["Rel"] = x["Rel"] * np.float32(16)   # exact in bf16; a wrong row of the table shifts a score by about its own size
    run_case(w, x, scaled=True)


# the bias table of a token tile formed out of LDS (up to 96 ids) and as a ring of 128: the last and first k of either, a whole
# turn of the ring and many, ids that end inside a block of 16, levels narrower than a pair of chunks (k = 6), the largest
# numbers of ids (629: forward only, the query side takes up to 512), sequences of their own lengths (causal: the ring;
# bidirectional with up to about 300 ids: out of LDS, masked at once)
@pytest.mark.parametrize("n,k,causal,lengths", [
    (4096, 10, True, None), (4096, 11, True, None), (1024, 5, False, None), (1024, 6, False, None), (256, 63, False, None), (8192, 15, True, None),
    (512, 33, False, [512, 400, 17]), (1024, 20, True, [1000, 1024]), (2048, 45, False, None), (2048, 61, False, None), (64, 31, False, [40, 64, 1])])
def test_bias_table_whole_and_as_a_ring(n, k, causal, lengths):
    # (a wrong row of the table, 16 times the usual size, shifts a score by about its own size)
    # (more than 1024 tiles: with fewer the forward stages its table)
    H = 16384 // (n * (len(lengths) if lengths else 1)) + 1
    run_token_tiles(n, k, causal, lengths, rel_times=16, query_side=(n, k) != (2048, 61), H=H)


# bidirectional sequences that end before n: the nodes past their end are masked as the blocks of ids enter the ring.  n =
# 256, k = 240: a last tile's second pair of chunks goes from the left side of level 0 to the left side of level 1, over
# more ids than the ring holds, all of them right-side ids past the end; masks of ids that the ring no longer holds would fall
# on the level-1 nodes.  Those (every span node) have values eight times as large here, so that a lost edge shows: the 7 of 250
# edges that token 250 then loses change `out` by sqrt(7) * 8 / 250 = 0.08 and lse by 0.03.
@pytest.mark.parametrize("n,k,lengths", [(256, 240, [255, 250]), (256, 300, [255, 241]), (1024, 60, [1024, 700]), (1024, 60, [1000, 33])])
def test_ring_masks_past_the_end_of_a_sequence(n, k, lengths):
    run_token_tiles(n, k, False, lengths, v_times=8)


def run_token_tiles(n, k, causal, lengths, p=0.0, v_times=1, rel_times=1, query_side=True, H=2):
    """Forward and backward against the oracle with values of span nodes and a table that are larger than usual (powers
    of two: exact in bf16), so that a lost edge or a wrong row of the table shows; the token rows must run on tiles
    (query_side: also in the backward)."""
    say("token tiles", n, k, causal, lengths, p)
    B = len(lengths) if lengths else 1
    w = Workload("token_tiles", 13, n, k, causal, B, H, 64, "bf16", True)
    x = make_inputs(w)
    x["V"][:, :, n:] *= np.float32(v_times)
    x["Rel"] = x["Rel"] * np.float32(rel_times)
    seed = 20191104 + n + k
    drop = (p, seed) if p > 0 else None
    g = bpt.bpt_build_graph(n, k, causal)
    Q, K, V, dO, R = (to_dev(x[k_], "bf16") for k_ in ("Q", "K", "V", "dO", "Rel"))
    lens_d = torch.tensor(lengths, dtype=torch.int32, device="cuda") if lengths else None
    bpt.bpt_profile_enable(True)
    out_d, lse_d = bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale, seq_len=lens_d, dropout=drop)
    grads = bpt.bpt_attn_bwd(g, Q, K, V, R, lse_d, dO, scale=w.scale, seq_len=lens_d, dropout=drop)
    torch.cuda.synchronize()
    ran = set(bpt.bpt_profile_report())
    bpt.bpt_profile_enable(False)
    assert "fwd_tile_kernel" in ran and "fwd_kernel" not in ran, ran
    assert ("bwd_q_tile_kernel" in ran) == query_side and ("bwd_q_kernel" in ran) == (not query_side), ran
    ll = lengths if lengths else [n] * B
    o, l, _ = oracle.attn_fwd_lengths(n, k, causal, ll, x["Q"], x["K"], x["V"], x["Rel"], w.scale, dropout=p, seed=seed)
    refs = oracle.attn_bwd_lengths(n, k, causal, ll, x["Q"], x["K"], x["V"], x["Rel"], x["dO"], w.scale, dropout=p, seed=seed)
    res = {}
    for name, got_t, ref in zip(("out", "lse", "dQ", "dK", "dV", "d_rel"), (out_d, lse_d) + tuple(grads), (o, l) + refs):
        got = host(got_t)
        assert np.isfinite(got).all(), name
        res[name] = (float(np.abs(got - ref).max()), tol_for("bf16", ref, scaled=True) / ((1.0 - p) if name == "out" else 1.0))
    say("   max-abs errors", {k_: float("%.3g" % v[0]) for k_, v in res.items()})
    for name, (err, tol) in res.items():
        assert err <= tol, (name, err, tol)
    g.destroy()


# graphs whose ids are too many for a staged table (more than about 300) and too far apart within a pair of chunks for the
# ring: the whole table out of memory, by pairs or (bidirectional sequences that end before n) at once.  459, 359, 436, 289 and
# 345 ids, k = 45: the ring without lengths, out of memory with them; the last: the largest number of ids, 479
@pytest.mark.parametrize("n,k,causal,lengths,p", [
    (512, 80, False, None, 0.0), (512, 80, False, [512, 300, 33], 0.0), (512, 80, False, [400, 511], 0.1), (1024, 120, True, None, 0.0),
    (1024, 120, True, [1000, 77], 0.0), (2048, 100, True, None, 0.2), (512, 127, True, None, 0.0), (256, 87, False, [255, 100, 1], 0.0),
    (512, 45, False, [512, 300, 33], 0.0), (512, 45, False, [450, 511], 0.1), (512, 88, False, [511], 0.0)])
def test_token_tiles_with_the_table_out_of_memory(n, k, causal, lengths, p):
    run_token_tiles(n, k, causal, lengths, p, rel_times=16)


@pytest.mark.parametrize("name", FULL)
def test_full_size_configuration(name):
    # configurations 2-5 at their full sizes, every output element against the oracle
    run_case(WORKLOADS[name])


def test_sequence_of_262144_tokens():
    # four times the longest benchmark sequence, one (batch, head): 19 levels, every output element
    run_case(Workload("long", 26, 262144, 2, True, 1, 1, 64, "bf16", True))


def run_lengths_case(w: Workload, lengths, poison=50.0):
    """A batch whose b-th sequence has lengths[b] <= n tokens: GPU (seq_len argument) against the oracle
    run per batch entry on the graph of that length.  Input rows of nodes that are not kept are
    multiplied by `poison`: they must not matter, and their outputs must be zero."""
    say("lengths case", w, list(lengths))
    assert len(lengths) == w.B
    x = make_inputs(w)
    for b, length in enumerate(lengths):
        if length >= 1:
            gone = np.flatnonzero(np.diff(oracle.build_graph_len(w.n, int(length), w.k, w.causal).row_ptr) == 0)
        else:
            gone = np.arange(2 * w.n - 1)
        for key in ("Q", "K", "V", "dO"):
            x[key][b][:, gone] *= np.float32(poison)
            if w.dtype == "bf16":                             # keep the values bf16-representable
                x[key][b][:, gone] = torch.from_numpy(x[key][b][:, gone]).to(torch.bfloat16).float().numpy()
    g = bpt.bpt_build_graph(w.n, w.k, w.causal)
    Q, K, V, dO, R = (to_dev(x[k], w.dtype) for k in ("Q", "K", "V", "dO", "Rel"))
    lens_d = torch.tensor(list(lengths), dtype=torch.int32, device="cuda")
    out_d, lse_d = bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale, seq_len=lens_d)
    grads = bpt.bpt_attn_bwd(g, Q, K, V, R, lse_d, dO, scale=w.scale, seq_len=lens_d)
    torch.cuda.synchronize()
    live = [b for b, length in enumerate(lengths) if length >= 1]
    ref = {k: np.zeros(x["Q"].shape) for k in ("out", "dQ", "dK", "dV")}
    ref["lse"] = np.zeros(x["Q"].shape[:3])
    ref["d_rel"] = np.zeros(x["Rel"].shape)
    if live:
        sub = {k: np.ascontiguousarray(x[k][live]) for k in ("Q", "K", "V", "dO")}
        ll = [lengths[b] for b in live]
        o, l, _ = oracle.attn_fwd_lengths(w.n, w.k, w.causal, ll, sub["Q"], sub["K"], sub["V"], x["Rel"], w.scale)
        dq, dk, dv, dr = oracle.attn_bwd_lengths(w.n, w.k, w.causal, ll, sub["Q"], sub["K"], sub["V"], x["Rel"],
                                                 sub["dO"], w.scale)
        ref["out"][live], ref["lse"][live], ref["dQ"][live], ref["dK"][live], ref["dV"][live] = o, l, dq, dk, dv
        ref["d_rel"] = dr
    res = {}
    for name, got_t in zip(("out", "lse", "dQ", "dK", "dV", "d_rel"), (out_d, lse_d) + tuple(grads)):
        got = host(got_t)
        assert np.isfinite(got).all(), name
        err = float(np.abs(got - ref[name]).max())
        res[name] = err
        assert err <= TOL[w.dtype], (name, err)
    # rows of nodes that are not kept: exact zeros
    for b, length in enumerate(lengths):
        deg = np.diff(oracle.build_graph_len(w.n, max(int(length), 1), w.k, w.causal).row_ptr)
        gone = np.flatnonzero(deg == 0) if length >= 1 else np.arange(2 * w.n - 1)
        for name, got_t in zip(("out", "lse", "dQ", "dK", "dV"), (out_d, lse_d) + tuple(grads[:3])):
            assert float(host(got_t)[b][:, gone].__abs__().max(initial=0.0)) == 0.0, (name, b)
    say("   max-abs errors", {k: float("%.3g" % v) for k, v in res.items()})
    g.destroy()


LENGTHS = [
    # fp32: gather kernels
    ("f32", 8, 1, False, 1, [8, 1, 5, 3]), ("f32", 64, 2, False, 2, [64, 1, 37, 17]), ("f32", 256, 3, True, 1, [100, 256, 2]),
    ("f32", 2048, 5, False, 1, [1500, 700]),
    # bf16 below the tile sizes, and around the switches of the tile kernels
    ("bf16", 8, 2, False, 1, [5, 8]), ("bf16", 16, 1, False, 2, [16, 9, 1]), ("bf16", 32, 1, True, 1, [31, 17, 32]),
    ("bf16", 64, 2, False, 1, [33, 64, 2, 48]),
    # bf16 tile kernels: ragged ends inside a tile, a whole sequence of one token, an empty one
    ("bf16", 512, 4, False, 2, [512, 300, 33, 1, 0]), ("bf16", 1024, 3, True, 2, [1000, 17, 1024]),
    ("bf16", 2048, 16, False, 1, [2047, 1025]), ("bf16", 4096, 8, True, 1, [3000, 4096, 129]),
    ("bf16", 4096, 40, False, 1, [2500]),
]


@pytest.mark.parametrize("dtype,n,k,causal,H,lengths", LENGTHS)
def test_sequences_of_different_lengths(dtype, n, k, causal, H, lengths):
    w = Workload("lengths", 21, n, k, causal, len(lengths), H, 64, dtype, True)
    run_lengths_case(w, lengths)


def test_lengths_of_a_batch_of_300():
    # more entries than the token-tile kernels number in closed form (256): the walk over all tiles with its
    # skips takes over; and 200, which they do number
    for B in (300, 200):
        rng = np.random.default_rng(300 + B)
        lengths = [int(v) for v in rng.integers(0, 65, size=B)]
        run_lengths_case(Workload("batch%d" % B, 23, 64, 2, False, B, 1, 64, "bf16", True), lengths)


def test_lengths_with_node_major_memory_and_many_ids():
    # [B,N,H,D] memory through the strides, and a density whose key tiles park table operands in LDS
    w = Workload("lengths_dense", 23, 1024, 64, False, 2, 2, 64, "bf16", True)
    lengths = [700, 1024]
    x = make_inputs(w)
    g = bpt.bpt_build_graph(w.n, w.k, w.causal)
    dev = {}
    for key in ("Q", "K", "V", "dO"):
        dev[key] = to_dev(x[key], w.dtype).permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    R = to_dev(x["Rel"], w.dtype)
    lens_d = torch.tensor(lengths, dtype=torch.int32, device="cuda")
    out_d, lse_d = bpt.bpt_attn_fwd(g, dev["Q"], dev["K"], dev["V"], R, scale=w.scale, seq_len=lens_d)
    grads = bpt.bpt_attn_bwd(g, dev["Q"], dev["K"], dev["V"], R, lse_d, dev["dO"], scale=w.scale, seq_len=lens_d)
    torch.cuda.synchronize()
    o, l, _ = oracle.attn_fwd_lengths(w.n, w.k, w.causal, lengths, x["Q"], x["K"], x["V"], x["Rel"], w.scale)
    refs = oracle.attn_bwd_lengths(w.n, w.k, w.causal, lengths, x["Q"], x["K"], x["V"], x["Rel"], x["dO"], w.scale)
    for name, got_t, ref in zip(("out", "lse", "dQ", "dK", "dV", "d_rel"), (out_d, lse_d) + tuple(grads), (o, l) + refs):
        err = float(np.abs(host(got_t) - ref).max())
        assert err <= TOL[w.dtype], (name, err)
    g.destroy()


@pytest.mark.parametrize("dtype,n,k,causal,H,lengths", [
    ("bf16", 512, 4, False, 2, [512, 300, 33, 1, 0]), ("bf16", 4096, 8, True, 1, [3000, 4096, 129]),
    ("bf16", 2048, 16, False, 1, [2047, 1025]), ("bf16", 8192, 8, True, 2, [1332, 7532]), ("f32", 256, 3, True, 1, [100, 256, 2]),
])
def test_rows_of_unkept_nodes_left_unwritten(dtype, n, k, causal, H, lengths):
    # bpt_shape_t.leave_unkept: the rows of kept nodes are those of the zero-filling calls bit for bit, and so is
    # d_rel; no NaN or Inf appears anywhere (the buffers start from a finite pattern).  With the matrix-core
    # kernels (bf16) the rows of whole tiles and blocks past the end of a sequence still hold that pattern.
    say("leave unkept", dtype, n, k, causal, H, lengths)
    w = Workload("unkept", 28, n, k, causal, len(lengths), H, 64, dtype, True)
    x = make_inputs(w)
    g = bpt.bpt_build_graph(n, k, causal)
    Q, K, V, dO, R = (to_dev(x[k_], dtype) for k_ in ("Q", "K", "V", "dO", "Rel"))
    lens_d = torch.tensor(list(lengths), dtype=torch.int32, device="cuda")
    out0, lse0 = bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale, seq_len=lens_d)
    grads0 = bpt.bpt_attn_bwd(g, Q, K, V, R, lse0, dO, scale=w.scale, seq_len=lens_d)
    mark = 7.0
    out1 = torch.full_like(Q, mark)
    lse1 = torch.full(Q.shape[:3], mark, dtype=torch.float32, device="cuda")
    grads1 = tuple(torch.full(Q.shape, mark, dtype=torch.float32, device="cuda") for _ in range(3)) + (
        torch.full(R.shape, mark, dtype=torch.float32, device="cuda"),)
    bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale, seq_len=lens_d, out=out1, lse=lse1, leave_unkept=True)
    lse_in = torch.where(lse1 == mark, torch.zeros_like(lse1), lse1)   # the backward reads lse of kept rows only
    bpt.bpt_attn_bwd(g, Q, K, V, R, lse_in, dO, scale=w.scale, seq_len=lens_d, grads=grads1, leave_unkept=True)
    torch.cuda.synchronize()
    assert torch.equal(grads0[3], grads1[3])          # d_rel does not depend on the option
    untouched = 0
    for b, length in enumerate(lengths):
        deg = np.diff(oracle.build_graph_len(n, max(int(length), 1), k, causal).row_ptr)
        kept = torch.from_numpy(np.flatnonzero(deg > 0) if length >= 1 else np.zeros(0, dtype=np.int64)).cuda()
        gone = np.flatnonzero(deg == 0) if length >= 1 else np.arange(2 * n - 1)
        for name, a0, a1 in zip(("out", "lse", "dQ", "dK", "dV"), (out0, lse0) + tuple(grads0[:3]), (out1, lse1) + tuple(grads1[:3])):
            assert torch.equal(a0[b][:, kept], a1[b][:, kept]), (name, b)
            assert bool(torch.isfinite(a1[b].float()).all()), (name, b)
        # nodes of whole token tiles / span blocks past the end: nothing was written there
        far = torch.from_numpy(gone[(gone >= ((length + 31) // 32) * 32) & (gone < n)]).cuda()
        if dtype == "bf16" and n >= 64 and len(far):
            untouched += int(far.numel())
            for name, a1 in zip(("out", "dQ", "dK", "dV"), (out1,) + tuple(grads1[:3])):
                assert bool((a1[b][:, far].float() == mark).all()), (name, b)
    if dtype == "bf16" and min(lengths) + 64 <= n:
        assert untouched > 0
    g.destroy()


def test_lengths_equal_to_n_change_nothing():
    w = Workload("full_lengths", 22, 1024, 4, False, 2, 2, 64, "bf16", True)
    x = make_inputs(w)
    g = bpt.bpt_build_graph(w.n, w.k, w.causal)
    Q, K, V, dO, R = (to_dev(x[k], w.dtype) for k in ("Q", "K", "V", "dO", "Rel"))
    lens_d = torch.full((w.B,), w.n, dtype=torch.int32, device="cuda")
    a = bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale)
    b = bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale, seq_len=lens_d)
    ga = bpt.bpt_attn_bwd(g, Q, K, V, R, a[1], dO, scale=w.scale)
    gb = bpt.bpt_attn_bwd(g, Q, K, V, R, b[1], dO, scale=w.scale, seq_len=lens_d)
    for s, t in zip(a + tuple(ga[:3]), b + tuple(gb[:3])):
        assert torch.equal(s, t)
    # d_rel is a sum over the whole batch; with seq_len the work is spread over the workgroups in
    # another order, so its partial sums round differently
    assert float((ga[3] - gb[3]).abs().max()) <= 1e-3 * float(ga[3].abs().max())
    g.destroy()


def test_random_small_configurations():
    # seeded draws over sizes, densities, direction, batch shape, dtype and lengths: every kernel family
    # and every switch between them gets hit with shapes nobody picked by hand
    rng = np.random.default_rng(20191111)
    for case in range(24):
        n = int(2 ** rng.integers(1, 11))
        k = int(rng.integers(1, 2 * n + 2)) if rng.random() < 0.3 else int(rng.integers(1, 12))
        causal = bool(rng.integers(0, 2))
        B, H = int(rng.integers(1, 4)), int(rng.integers(1, 4))
        dtype = "bf16" if rng.random() < 0.7 else "f32"
        w = Workload("random%d" % case, 30 + case, n, k, causal, B, H, 64, dtype, True)
        if rng.random() < 0.5:
            lengths = [int(rng.integers(0 if rng.random() < 0.1 else 1, n + 1)) for _ in range(B)]
            run_lengths_case(w, lengths)
        else:
            run_case(w)


DROPOUT = [
    ("f32", 64, 2, False, 2, 2, 0.1, None), ("f32", 256, 3, True, 1, 2, 0.5, None),
    ("bf16", 512, 4, False, 2, 2, 0.1, None), ("bf16", 2048, 8, True, 1, 2, 0.3, None),
    ("bf16", 1024, 5, False, 2, 1, 0.2, [1000, 300]), ("bf16", 4096, 40, False, 1, 1, 0.1, None),
    ("bf16", 2048, 16, True, 2, 1, 0.25, [2048, 777]), ("bf16", 8192, 8, True, 1, 1, 0.1, None),
]


@pytest.mark.parametrize("dtype,n,k,causal,B,H,p,lengths", DROPOUT)
def test_dropout_on_attention_weights(dtype, n, k, causal, B, H, p, lengths):
    # the same counter-based mask on both sides: an edge is dropped on the GPU iff the oracle drops it
    say("dropout", dtype, n, k, causal, B, H, p, lengths)
    w = Workload("dropout", 25, n, k, causal, B, H, 64, dtype, True)
    seed = 20191104 + n
    x = make_inputs(w)
    g = bpt.bpt_build_graph(n, k, causal)
    Q, K, V, dO, R = (to_dev(x[k_], dtype) for k_ in ("Q", "K", "V", "dO", "Rel"))
    lens = lengths if lengths is not None else [n] * B
    lens_d = torch.tensor(lens, dtype=torch.int32, device="cuda") if lengths is not None else None
    out_d, lse_d = bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale, seq_len=lens_d, dropout=(p, seed))
    grads = bpt.bpt_attn_bwd(g, Q, K, V, R, lse_d, dO, scale=w.scale, seq_len=lens_d, dropout=(p, seed))
    torch.cuda.synchronize()
    o, l, _ = oracle.attn_fwd_lengths(n, k, causal, lens, x["Q"], x["K"], x["V"], x["Rel"], w.scale, dropout=p, seed=seed)
    refs = oracle.attn_bwd_lengths(n, k, causal, lens, x["Q"], x["K"], x["V"], x["Rel"], x["dO"], w.scale, dropout=p,
                                   seed=seed)
    res = {}
    for name, got_t, ref in zip(("out", "lse", "dQ", "dK", "dV", "d_rel"), (out_d, lse_d) + tuple(grads), (o, l) + refs):
        got = host(got_t)
        assert np.isfinite(got).all(), name
        res[name] = float(np.abs(got - ref).max())
        # the absolute tolerance is that of a convex combination of value rows; inverted dropout multiplies a row of
        # `out` (rounded to the tensors' dtype) by up to 1/(1-p), and the rounding step with it
        tol = TOL[dtype] / (1.0 - p) if name == "out" else TOL[dtype]
        assert res[name] <= tol, (name, res[name])
    # and it is a different result from the one without dropout
    out0, _ = bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale, seq_len=lens_d)
    assert float((out0.float() - out_d.float()).abs().max()) > 0.05
    say("   max-abs errors", {k_: float("%.3g" % v) for k_, v in res.items()})
    g.destroy()


def test_autograd_function_returns_the_library_gradients():
    w = Workload("autograd", 24, 256, 3, False, 2, 2, 64, "f32", True)
    x = make_inputs(w)
    g = bpt.bpt_build_graph(w.n, w.k, w.causal)
    Q, K, V, R, dO = (to_dev(x[k], "f32") for k in ("Q", "K", "V", "Rel", "dO"))
    leaves = [t.clone().requires_grad_(True) for t in (Q, K, V, R)]
    out = bpt.graph_attention(g, *leaves, scale=w.scale)
    out.backward(dO)
    ref_out, lse = bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale)
    ref = bpt.bpt_attn_bwd(g, Q, K, V, R, lse, dO, scale=w.scale)
    assert torch.equal(out.detach(), ref_out)
    for leaf, r in zip(leaves, ref):
        assert torch.equal(leaf.grad, r)
    g.destroy()


@pytest.mark.parametrize("dtype,n,k,causal,B,H,q_times,rel_std", [
    ("bf16", 1024, 4, False, 2, 2, 4.0, 0.5), ("bf16", 1024, 4, True, 2, 2, 8.0, 0.5), ("bf16", 4096, 8, True, 1, 2, 8.0, 0.25),
    ("f32", 512, 3, False, 1, 2, 4.0, 0.5), ("f32", 512, 3, True, 1, 2, 8.0, 1.0),
])
def test_peaked_rows_and_a_large_relative_position_table(dtype, n, k, causal, B, H, q_times, rel_std):
    # scores with a deviation of 4..8 instead of 1 (most rows put nearly all their weight on one or two keys: lse up
    # to 48, and dS = w - delta p is a difference of nearly equal numbers) and a table as large as a trained one
    # (its terms are then a sizeable part of every score, of dQ and of d_rel).  Q is multiplied by a power of
    # two, which keeps its values exact in bf16; the table is rounded again after scaling.
    from paper_1911_04070_amd.workloads import REL_STD, round_to_bf16
    w = Workload("peaked", 9, n, k, causal, B, H, 64, dtype, True)
    x = make_inputs(w)
    x["Q"] = (x["Q"] * q_times).astype(np.float32)
    rel = (x["Rel"] * (rel_std / REL_STD)).astype(np.float32)
    x["Rel"] = round_to_bf16(rel)[0] if dtype == "bf16" else rel
    res = run_case(w, x=x, scaled=True)
    assert res["d_rel_max"] > 10.0   # the table's gradient is not small here


VISIBLE_TABLE = [
    # (n, k, causal, B, H, q_times, rel_std, lengths, dropout rate, must run rel_grad_tile_kernel)
    # up to 256 ids in use: (w, p) hand-over, d_rel kernel with two id groups, key tiles with 2..3 chunks of ids
    (4096, 8, False, 1, 2, 4.0, 0.5, None, 0.0, True),
    # more than 256 ids: d_rel kernel with four id groups, the forward's and the query side's bias as a ring
    (4096, 16, False, 1, 2, 8.0, 0.25, None, 0.0, True),
    (4096, 32, False, 1, 2, 4.0, 0.5, None, 0.0, True),
    # the character-level density: key tiles with 9 blocks of ids, five of them in registers at a time
    (8192, 64, True, 1, 1, 4.0, 0.5, None, 0.0, True),
    # the same variants with shorter sequences and with dropout on the weights
    (4096, 16, False, 2, 1, 4.0, 0.5, [3000, 4096], 0.0, True),
    (4096, 32, False, 1, 1, 4.0, 0.5, None, 0.2, True),
    (4096, 64, True, 1, 1, 8.0, 0.25, [2500], 0.1, True),
    # dense query side (at most 128 ids) with lengths and dropout at once
    (2048, 4, False, 2, 1, 4.0, 0.5, [2048, 1100], 0.15, False),
]


@pytest.mark.parametrize("n,k,causal,B,H,q_times,rel_std,lengths,p,hand_over", VISIBLE_TABLE)
def test_large_table_on_every_kernel_variant(n, k, causal, B, H, q_times, rel_std, lengths, p, hand_over):
    # With the task's table of deviation 0.02 the relative-position term of a score is smaller than the bf16
    # tolerance, so a kernel that dropped it would pass.  Here the table is as large as a trained one (its term has
    # a deviation of 1..2 per score) on graphs that select the kernel variants for many ids: the (w, p) hand-over
    # with its d_rel kernel (which also adds the table's part of dQ), table rows read from memory pair by pair,
    # key tiles with 3..9 chunks of ids -- alone, with shorter sequences and with dropout.
    from paper_1911_04070_amd.workloads import REL_STD, round_to_bf16
    say("visible table", n, k, causal, B, H, q_times, rel_std, lengths, p)
    w = Workload("visible", 12, n, k, causal, B, H, 64, "bf16", True)
    x = make_inputs(w)
    x["Q"] = (x["Q"] * q_times).astype(np.float32)
    x["Rel"] = round_to_bf16((x["Rel"] * (rel_std / REL_STD)).astype(np.float32))[0]
    seed = 20191104 + n + k
    drop = (p, seed) if p > 0 else None
    lens = lengths if lengths is not None else [n] * B
    lens_d = torch.tensor(lens, dtype=torch.int32, device="cuda") if lengths is not None else None
    g = bpt.bpt_build_graph(n, k, causal)
    Q, K, V, dO, R = (to_dev(x[k_], "bf16") for k_ in ("Q", "K", "V", "dO", "Rel"))
    bpt.bpt_profile_enable(True)
    out_d, lse_d = bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale, seq_len=lens_d, dropout=drop)
    grads = bpt.bpt_attn_bwd(g, Q, K, V, R, lse_d, dO, scale=w.scale, seq_len=lens_d, dropout=drop)
    torch.cuda.synchronize()
    ran = set(bpt.bpt_profile_report())
    bpt.bpt_profile_enable(False)
    assert {"fwd_tile_kernel", "bwd_q_tile_kernel"} <= ran, ran   # the matrix-core path
    assert ran & {"bwd_kv_tile_kernel", "bwd_kv_chain_kernel"}, ran
    assert ("rel_grad_tile_kernel" in ran) == hand_over, ran
    o, l, _ = oracle.attn_fwd_lengths(n, k, causal, lens, x["Q"], x["K"], x["V"], x["Rel"], w.scale, dropout=p, seed=seed)
    refs = oracle.attn_bwd_lengths(n, k, causal, lens, x["Q"], x["K"], x["V"], x["Rel"], x["dO"], w.scale, dropout=p,
                                   seed=seed)
    res = {}
    for name, got_t, ref in zip(("out", "lse", "dQ", "dK", "dV", "d_rel"), (out_d, lse_d) + tuple(grads), (o, l) + refs):
        got = host(got_t)
        assert np.isfinite(got).all(), name
        res[name] = float(np.abs(got - ref).max())
        res[name + "_max"] = float(np.abs(ref).max())
        tol = tol_for("bf16", ref, scaled=True) / ((1.0 - p) if name == "out" else 1.0)
        assert res[name] <= tol, (name, res[name], tol)
    say("   max-abs errors", {k_: float("%.3g" % v) for k_, v in res.items()})
    assert res["d_rel_max"] > 10.0
    # what the table contributes is far above the bound: with a zero table the forward differs by more than
    # ten times the tolerance, so a kernel without the term could not have passed
    out0, lse0 = bpt.bpt_attn_fwd(g, Q, K, V, torch.zeros_like(R), scale=w.scale, seq_len=lens_d, dropout=drop)
    assert float((lse0.double().cpu() - torch.from_numpy(l)).abs().max()) > 10 * tol_for("bf16", l, scaled=True)
    assert float((out0.float() - out_d.float()).abs().max()) > 0.2
    g.destroy()


@pytest.mark.parametrize("n,k,causal,step", [(512, 4, False, 1.0), (512, 4, False, 5.0), (2048, 16, True, 1.0), (1024, 24, False, 5.0),
                                             (512, 8, False, -1.0), (512, 80, False, 1.0)])
def test_scores_that_rise_along_a_row(n, k, causal, step):
    # the reference of a row's softmax moves with (or stays through) every pair of chunks: scores that rise (or fall) by
    # step / ln 2 powers of two per level of the key, on tables in LDS, as a ring and in memory
    w = Workload("rising", 15, n, k, causal, 1, 3, 64, "bf16", False)
    x = make_inputs(w)
    level = np.maximum(n.bit_length() - 1 - np.floor(np.log2(2 * n - 1 - np.arange(2 * n - 1))).astype(int), 0)
    x["Q"][..., 0] = 8.0                              # score = (8 * step * level + the other features) / 8
    x["K"][..., 0] = step * level
    run_case(w, x, scaled=True)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_zero_queries_and_zero_values(dtype):
    # degenerate rows: q = 0 makes every row uniform over its neighbours (lse = ln deg, dK = d_rel = 0);
    # v = 0 makes out, dP and with them dQ, dK and d_rel exactly zero
    w = Workload("zeros", 11, 512, 3, False, 2, 2, 64, dtype, True)
    x = make_inputs(w)
    x["Q"] = np.zeros_like(x["Q"])
    res = run_case(w, x=x)
    assert res["dK_max"] == 0.0 and res["d_rel_max"] == 0.0 and res["dK"] == 0.0 and res["d_rel"] == 0.0
    x = make_inputs(w)
    x["V"] = np.zeros_like(x["V"])
    res = run_case(w, x=x)
    assert res["out"] == 0.0 and res["dQ"] == 0.0 and res["dK"] == 0.0 and res["d_rel"] == 0.0


def test_scale_argument_and_default():
    w = Workload("scale", 10, 256, 2, False, 1, 2, 64, "f32", True)
    x = make_inputs(w)
    ref_g = oracle.build_graph(w.n, w.k, w.causal)
    g = bpt.bpt_build_graph(w.n, w.k, w.causal)
    Q, K, V, R = (to_dev(x[k], "f32") for k in ("Q", "K", "V", "Rel"))
    for scale, eff in ((None, 0.125), (0.05, 0.05)):
        out_d, lse_d = bpt.bpt_attn_fwd(g, Q, K, V, R, scale=scale)
        out_r, lse_r, _ = oracle.attn_fwd(ref_g, x["Q"], x["K"], x["V"], x["Rel"], eff)
        assert np.abs(host(out_d) - out_r).max() <= 1e-4
        assert np.abs(host(lse_d) - lse_r).max() <= 1e-4
    g.destroy()


def test_run_to_run_reproducibility():
    w = shrink(WORKLOADS["lm"], B=1, H=2, n=2048)
    x = make_inputs(w)
    g = bpt.bpt_build_graph(w.n, w.k, w.causal)
    Q, K, V, R, dO = (to_dev(x[k], "bf16") for k in ("Q", "K", "V", "Rel", "dO"))
    runs = []
    for _ in range(3):
        out, lse = bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale)
        grads = bpt.bpt_attn_bwd(g, Q, K, V, R, lse, dO, scale=w.scale)
        torch.cuda.synchronize()
        runs.append([t.clone() for t in (out, lse) + tuple(grads)])
    for other in runs[1:]:
        for name, a, b in zip(("out", "lse", "dQ", "dK", "dV", "d_rel"), runs[0], other):
            assert torch.equal(a, b), name                      # no atomics anywhere: bit-identical
    g.destroy()


BF16_GRADS = [
    # (n, k, causal, B, H, lengths, leave_unkept, node_major)
    (16, 1, False, 2, 2, None, False, False),              # gather kernels
    (1024, 4, False, 2, 2, None, False, False),            # token tiles with dense dS, key tiles chained
    (4096, 8, True, 1, 2, None, False, True),              # the language-model density, node-major memory
    (4096, 16, False, 1, 1, None, False, False),          # more than 128 ids: rel_grad_tile_kernel adds to dQ
    (2048, 40, False, 1, 1, None, False, False),          # key tiles that fetch table operands pair by pair
    (512, 4, False, 3, 2, [512, 300, 33], False, False),   # lengths, zero rows
    (4096, 8, True, 2, 1, [3000, 129], True, False),       # lengths, rows left unwritten
]


@pytest.mark.parametrize("n,k,causal,B,H,lengths,leave,node_major", BF16_GRADS)
def test_gradients_rounded_to_bf16(n, k, causal, B, H, lengths, leave, node_major):
    # bpt_shape_t.grad_dtype = BPT_BF16: dQ, dK, dV are the fp32 sums of the default call rounded to nearest even
    # once, bit for bit -- dQ also where a second kernel adds the relative-position part to it (graphs with more than 128
    # ids in use); d_rel does not depend on the option
    say("bf16 gradients", n, k, causal, B, H, lengths, leave, node_major)
    w = Workload("bf16_grads", 31, n, k, causal, B, H, 64, "bf16", True)
    x = make_inputs(w)
    g = bpt.bpt_build_graph(n, k, causal)
    if node_major:
        Q, K, V, dO = (to_dev(np.transpose(x[k_], (0, 2, 1, 3)), "bf16").transpose(1, 2) for k_ in ("Q", "K", "V", "dO"))
    else:
        Q, K, V, dO = (to_dev(x[k_], "bf16") for k_ in ("Q", "K", "V", "dO"))
    R = to_dev(x["Rel"], "bf16")
    lens_d = torch.tensor(lengths, dtype=torch.int32, device="cuda") if lengths else None
    out, lse = bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale, seq_len=lens_d)
    mark = 3.0
    g32 = tuple(torch.full_like(Q, mark, dtype=torch.float32) for _ in range(3)) + (torch.empty_like(R, dtype=torch.float32),)
    g16 = tuple(torch.full_like(Q, mark) for _ in range(3)) + (torch.empty_like(R, dtype=torch.float32),)
    bpt.bpt_attn_bwd(g, Q, K, V, R, lse, dO, scale=w.scale, seq_len=lens_d, leave_unkept=leave, grads=g32)
    bpt.bpt_attn_bwd(g, Q, K, V, R, lse, dO, scale=w.scale, seq_len=lens_d, leave_unkept=leave, grads=g16)
    torch.cuda.synchronize()
    assert g16[0].dtype == torch.bfloat16 and g16[0].stride() == Q.stride()
    assert torch.equal(g32[3], g16[3])
    for name, a32, a16 in zip(("dQ", "dK", "dV"), g32[:3], g16[:3]):
        assert torch.equal(a16, a32.to(torch.bfloat16)), name
    # the two-stage calls take the option too
    dq2, dk2, dv2 = (torch.full_like(Q, mark) for _ in range(3))
    ws = torch.empty(bpt.workspace_bytes(g, Q, w.scale)[1] + 256, dtype=torch.uint8, device="cuda")
    bpt.bpt_attn_bwd_query_side(g, Q, K, V, R, lse, dO, dq2, g16[3], ws, scale=w.scale, seq_len=lens_d, leave_unkept=leave)
    bpt.bpt_attn_bwd_key_side(g, Q, K, V, R, lse, dO, dk2, dv2, ws, scale=w.scale, seq_len=lens_d, leave_unkept=leave)
    torch.cuda.synchronize()
    assert torch.equal(dq2, g16[0]) and torch.equal(dk2, g16[1]) and torch.equal(dv2, g16[2])
    with pytest.raises(ValueError):                      # all three of one type
        bpt.bpt_attn_bwd(g, Q, K, V, R, lse, dO, scale=w.scale, grads=(g16[0], g32[1], g32[2], g32[3]))
    g.destroy()


def test_backward_workspace_at_the_character_level_density():
    # the fp32 rows of dQ that bf16 gradients need for a while (64 MiB here) lie where the key side keeps its partial sums:
    # 4 x 8 heads on n = 8192, k = 64 take what they took when dQ was rounded twice
    g = bpt.bpt_build_graph(8192, 64, True)
    Q = torch.empty((4, 8, g.num_nodes, 64), dtype=torch.bfloat16, device="cuda")
    assert bpt.workspace_bytes(g, Q)[1] <= 975700224
    g.destroy()


def test_bf16_gradients_are_for_bf16_tensors():
    g = bpt.bpt_build_graph(64, 2, False)
    Q = torch.zeros(1, 1, g.num_nodes, 64, device="cuda")
    R = torch.zeros(g.num_levels, g.rel_width, 64, device="cuda")
    out, lse = bpt.bpt_attn_fwd(g, Q, Q, Q, R)
    with pytest.raises(ValueError):
        bpt.bpt_attn_bwd(g, Q, Q, Q, R, lse, Q, bf16_grads=True)
    shp = bpt._shape_of(g, Q, None, bf16_grads=True)      # the C side refuses the combination as well
    L = bpt.load_library()
    assert L.bpt_attn_bwd_workspace(g.handle, __import__("ctypes").byref(shp)) == 2 ** 64 - 1
    g.destroy()


def test_invalid_arguments_on_device():
    g = bpt.bpt_build_graph(64, 2, False)
    Q = torch.zeros(1, 1, g.num_nodes, 64, device="cuda")
    R = torch.zeros(g.num_levels, g.rel_width, 64, device="cuda")
    with pytest.raises(ValueError):
        bpt.bpt_attn_fwd(g, Q[:, :, :-1], Q[:, :, :-1], Q[:, :, :-1], R)
    Q32 = torch.zeros(1, 1, g.num_nodes, 32, device="cuda")
    R32 = torch.zeros(g.num_levels, g.rel_width, 32, device="cuda")
    with pytest.raises(bpt.BptError) as e:
        bpt.bpt_attn_fwd(g, Q32, Q32, Q32, R32)
    assert e.value.status == bpt.BPT_ERR_UNSUPPORTED
    g.destroy()


def test_forward_and_backward_replay_from_a_captured_graph():
    # the calls only launch kernels on the caller's stream (no allocation, no synchronisation, no memset
    # node), so a step can be captured once and replayed: every replay, with new inputs in the same
    # buffers and eager work of the program in between, gives the bits of the eager call
    w = Workload("capture", 27, 2048, 4, True, 2, 2, 64, "bf16", True)
    g = bpt.bpt_build_graph(w.n, w.k, w.causal)
    x = make_inputs(w)
    Q, K, V, dO, R = (to_dev(x[k_], "bf16") for k_ in ("Q", "K", "V", "dO", "Rel"))
    out = torch.empty_like(Q)
    lse = torch.empty(Q.shape[:3], dtype=torch.float32, device="cuda")
    grads = tuple(torch.empty(Q.shape, dtype=torch.float32, device="cuda") for _ in range(3)) + (
        torch.empty(R.shape, dtype=torch.float32, device="cuda"),)
    fws, bws = bpt.workspace_bytes(g, Q, w.scale)
    ws_f = torch.empty(max(fws, 256), dtype=torch.uint8, device="cuda")
    ws_b = torch.empty(max(bws, 256), dtype=torch.uint8, device="cuda")

    def step():
        bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale, out=out, lse=lse, workspace=ws_f)
        bpt.bpt_attn_bwd(g, Q, K, V, R, lse, dO, scale=w.scale, grads=grads, workspace=ws_b)

    step()                                   # first use of every kernel outside the capture
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        graph.capture_begin()
        step()
        graph.capture_end()
    torch.cuda.synchronize()
    gen = torch.Generator(device="cuda").manual_seed(5)
    for replay in range(3):
        for t in (Q, K, V, dO):              # new inputs in the captured buffers
            t.copy_(torch.randn(t.shape, device="cuda", generator=gen).to(t.dtype))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = [out.clone(), lse.clone()] + [t.clone() for t in grads]
        step()                               # eager, same buffers
        torch.cuda.synchronize()
        for name, a, b in zip(("out", "lse", "dQ", "dK", "dV", "d_rel"), got, [out, lse] + list(grads)):
            assert torch.equal(a, b), (replay, name)
    g.destroy()


@pytest.mark.parametrize("n,k,causal,B,lengths,leave", [
    (256, 3, False, 2, None, False),             # dQ complete in the tile kernel
    (2048, 16, False, 1, None, False),           # more than 128 ids: the relative-position part is added by a second kernel
    (2048, 16, False, 3, [1040, 17, 2048], False), (2048, 16, False, 3, [1040, 17, 1], True),
])
def test_bf16_gradients_are_rounded_once(n, k, causal, B, lengths, leave):
    # whichever kernels form dQ, the fp32 sum is rounded once: bit for bit the fp32 call's result rounded
    say("bf16 gradients, one rounding", n, k, causal, lengths, leave)
    w = Workload("bf16_once", 32, n, k, causal, B, 1, 64, "bf16", True)
    x = make_inputs(w)
    g = bpt.bpt_build_graph(n, k, causal)
    Q, K, V, R, dO = (to_dev(x[k_], "bf16") for k_ in ("Q", "K", "V", "Rel", "dO"))
    lens_d = torch.tensor(lengths, dtype=torch.int32, device="cuda") if lengths else None
    _, lse = bpt.bpt_attn_fwd(g, Q, K, V, R, seq_len=lens_d)
    g32 = tuple(torch.full_like(Q, 3.0, dtype=torch.float32) for _ in range(3)) + (torch.empty_like(R, dtype=torch.float32),)
    g16 = tuple(torch.full_like(Q, 3.0) for _ in range(3)) + (torch.empty_like(R, dtype=torch.float32),)
    bpt.bpt_attn_bwd(g, Q, K, V, R, lse, dO, grads=g32, seq_len=lens_d, leave_unkept=leave)
    bpt.bpt_attn_bwd(g, Q, K, V, R, lse, dO, grads=g16, seq_len=lens_d, leave_unkept=leave)
    torch.cuda.synchronize()
    for name, a32, a16 in zip(("dQ", "dK", "dV"), g32, g16):
        assert torch.equal(a16, a32.to(torch.bfloat16)), name
    if not leave:   # and what autograd hands out is that
        leaves = [t.clone().requires_grad_(True) for t in (Q, K, V, R)]
        bpt.graph_attention(g, *leaves, seq_len=lens_d).backward(dO)
        for leaf, a32 in zip(leaves, g32):
            assert torch.equal(leaf.grad, a32.to(torch.bfloat16))
    g.destroy()
