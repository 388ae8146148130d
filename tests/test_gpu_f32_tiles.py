"""fp32 tensors on the matrix cores, against the oracle, at the sizes where their tiles change."""
import numpy as np
import pytest

from paper_1911_04070_amd import binding as bpt
from paper_1911_04070_amd.workloads import Workload, make_inputs
from test_gpu_parity import run_case

pytestmark = pytest.mark.gpu

# (n, k, causal, B, H, ids token rows use): one tile with fewer chunks than wavefronts, with and without long span rows (more
# than 64 tokens, and more than 512: those have partial results), ids that end on and behind a block of 16, the last and first
# numbers of ids of the query side's variants (96, 192, 384; above that its gather kernel), tiles that several workgroups
# walk (more than 512) and key tiles cut into several tasks
CASES = [(16, 1, False, 1, 3, 15), (16, 30, True, 2, 1, 16), (32, 3, True, 1, 2, 14), (64, 5, False, 2, 2, 43), (128, 4, True, 1, 3, 25),
         (256, 8, False, 1, 2, 89), (512, 7, False, 1, 2, 99), (256, 24, False, 1, 2, 171), (1024, 44, True, 1, 1, 203),
         (1024, 25, False, 1, 1, 275), (512, 58, False, 1, 1, 381), (512, 59, False, 1, 1, 385), (1024, 3, True, 3, 4, 34),
         (4096, 4, False, 1, 2, None)]


@pytest.mark.parametrize("n,k,causal,B,H,ids,layout", [c + ("bhnd",) for c in CASES] + [CASES[3] + ("bnhd",), CASES[6] + ("bnhd",)])
def test_fp32_tiles(n, k, causal, B, H, ids, layout):
    w = Workload("f32_tiles", 14, n, k, causal, B, H, 64, "f32", True)
    x = make_inputs(w)
    x["Rel"] = x["Rel"] * np.float32(16)   # a wrong row of the table shifts a score by about its own size
    if ids is not None:
        g = bpt.bpt_build_graph(n, k, causal)
        row_ptr, _, rel = g.csr_to_host()
        assert len(np.unique(rel[:row_ptr[n]])) == ids
        g.destroy()
    bpt.bpt_profile_enable(True)
    run_case(w, x, layout=layout, scaled=True)
    ran = set(bpt.bpt_profile_report())
    bpt.bpt_profile_enable(False)
    tiles = {"bwd_q_f32_tile_kernel", "bwd_kv_f32_tile_kernel"}
    assert "fwd_f32_tile_kernel" in ran and "fwd_kernel" not in ran, ran
    assert tiles <= ran if ids is None or ids <= 384 else not tiles & ran, ran


@pytest.mark.parametrize("n,k,causal,key_tiles", [(16, 3966, False, True), (16, 3967, False, False), (64, 17000, True, False)])
def test_more_orders_than_the_key_side_holds(n, k, causal, key_tiles):
    # few ids in use, but 2 k + 3 orders per level: up to 7936 in the key side's LDS, the gather kernels beyond
    w = Workload("f32_tiles", 14, n, k, causal, 1, 2, 64, "f32", True)
    bpt.bpt_profile_enable(True)
    run_case(w, make_inputs(w), scaled=True)
    ran = set(bpt.bpt_profile_report())
    bpt.bpt_profile_enable(False)
    assert ("bwd_kv_f32_tile_kernel" in ran) == key_tiles and ("bwd_kv_kernel" in ran) != key_tiles, ran
