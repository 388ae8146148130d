"""Span rows above the blocks of 32 tokens (bf16): rows finished by a workgroup of four blocks, partial results of four blocks
added up or kept apart, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_04070_amd import binding as bpt
from paper_1911_04070_amd.workloads import Workload, make_inputs
from test_gpu_parity import host, say, to_dev, tol_for

pytestmark = pytest.mark.gpu

# (n, lengths, H, dropout): workgroups that serve two sequences of two blocks, the last of them half empty; trees that end at
# the workgroup's level and one above it; sequences that end on, behind and before an edge of blocks and workgroups; both
# sides of the size from which the forward adds four blocks up (2048); rows of more and fewer than 16 partial results
CASES = [(64, [64, 33, 31], 1, 0.0), (128, [128, 96, 65, 1], 1, 0.0), (256, [256, 129, 128], 2, 0.0), (1024, [1024, 700], 1, 0.0),
         (2048, [2048, 1409, 130], 1, 0.0), (2048, [2048, 1024], 1, 0.2), (4096, [4096, 2081], 1, 0.0)]


@pytest.mark.parametrize("n,lengths,H,p", CASES)
def test_span_rows_of_workgroups(n, lengths, H, p):
    say("span rows", n, lengths, H, p)
    w = Workload("span_groups", 15, n, 2, False, len(lengths), H, 64, "bf16", True)
    x = make_inputs(w)
    x["Q"] = (x["Q"] * 4).astype(np.float32)   # peaked weights: a row that misses a block misses what it consists of
    lens = torch.tensor(lengths, dtype=torch.int32, device="cuda")
    drop = (p, 7) if p > 0 else None
    g = bpt.bpt_build_graph(n, 2, False)
    Q, K, V, dO, R = (to_dev(x[key], "bf16") for key in ("Q", "K", "V", "dO", "Rel"))
    bpt.bpt_profile_enable(True)
    out, lse = bpt.bpt_attn_fwd(g, Q, K, V, R, scale=w.scale, seq_len=lens, dropout=drop)
    grads = bpt.bpt_attn_bwd(g, Q, K, V, R, lse, dO, scale=w.scale, seq_len=lens, dropout=drop)
    torch.cuda.synchronize()
    ran = set(bpt.bpt_profile_report())
    bpt.bpt_profile_enable(False)
    assert ("fwd_span_merge_kernel" in ran) == ("bwd_q_span_merge_kernel" in ran) == (n > 128), ran
    o, l, _ = oracle.attn_fwd_lengths(n, 2, False, lengths, x["Q"], x["K"], x["V"], x["Rel"], w.scale, dropout=p, seed=7)
    refs = oracle.attn_bwd_lengths(n, 2, False, lengths, x["Q"], x["K"], x["V"], x["Rel"], x["dO"], w.scale, dropout=p, seed=7)
    assert np.abs(o[:, :, -1]).max() > 0.2   # the root's row has something to lose
    for name, got, ref in zip(("out", "lse", "dQ", "dK", "dV"), (out, lse) + tuple(grads), (o, l) + refs):
        a = host(got)
        assert np.isfinite(a).all(), name
        assert np.abs(a - ref).max() <= tol_for("bf16", ref, scaled=True) / ((1.0 - p) if name == "out" else 1.0), name
    g.destroy()


@pytest.mark.parametrize("n,B,H", [(256, 112, 8), (512, 40, 8), (1024, 16, 8)])
@pytest.mark.parametrize("mixed", [False, True])
def test_rows_do_not_depend_on_the_batch(n, B, H, mixed):
    # forward below 2048 tokens: a large batch (20000 partial results and more) finishes levels 6 and 7 in the tile kernel, its
    # quarters leave all of them to the merge kernel; the rows have the same bits
    say("span rows, batch", n, B, H, mixed)
    levels, blocks = n.bit_length() - 1 - 5, n // 32
    assert B * H * blocks * levels >= 20000 > B // 4 * H * blocks * levels
    g = bpt.bpt_build_graph(n, 2, False)
    gen = torch.Generator(device="cuda").manual_seed(n)
    Q, K, V = (torch.randn(B, H, g.num_nodes, 64, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(3))
    R = torch.randn(g.num_levels, g.rel_width, 64, device="cuda", generator=gen).to(torch.bfloat16)
    lens = torch.randint(1, n + 1, (B,), dtype=torch.int32, device="cuda", generator=gen) if mixed else None
    out, lse = bpt.bpt_attn_fwd(g, Q, K, V, R, seq_len=lens)
    for b in range(0, B, B // 4):
        part = slice(b, b + B // 4)
        o, l = bpt.bpt_attn_fwd(g, Q[part].contiguous(), K[part].contiguous(), V[part].contiguous(), R,
                                seq_len=lens[part].contiguous() if mixed else None)
        assert torch.equal(out[part], o) and torch.equal(lse[part], l), b
    g.destroy()
