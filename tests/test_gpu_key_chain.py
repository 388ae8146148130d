"""Key side of the backward on chained tiles (bf16): tasks whose ids fit one chunk of 16 and tasks that need two."""
import numpy as np
import pytest

from paper_1911_04070_amd import binding as bpt
from paper_1911_04070_amd.workloads import Workload, make_inputs
from test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


# above the tokens ids go up to k (causal) or 2 k + 2: the last bidirectional k with one chunk there and the first with two,
# the largest causal ones; a tree whose token level stays below 16 as well, one where ids end on the last of a chunk
@pytest.mark.parametrize("n,k,causal", [(256, 6, False), (256, 7, False), (512, 8, True), (1024, 9, True), (64, 2, False), (128, 4, True)])
def test_ids_of_one_and_two_chunks(n, k, causal):
    w = Workload("key_chain", 16, n, k, causal, 1, 2, 64, "bf16", True)
    x = make_inputs(w)
    x["Rel"] = (x["Rel"] * np.float32(16)).astype(np.float32)   # a wrong row of the table shifts a score by about its own size
    x["Rel"] = (x["Rel"].view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)   # bf16 values
    bpt.bpt_profile_enable(True)
    run_case(w, x, scaled=True)
    ran = set(bpt.bpt_profile_report())
    bpt.bpt_profile_enable(False)
    assert "bwd_kv_chain_kernel" in ran, ran
