"""The blocks of batch graphs' tables (host code), on a stand-in for the HIP runtime whose queues advance when the test says so."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("table_pool") / "check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-D_GLIBCXX_ASSERTIONS", "-Wall", "-pthread", "-I", os.path.join(HERE, "table_pool"),
                           "-I", os.path.join(ROOT, "paper_1911_04070_amd", "csrc"), os.path.join(HERE, "table_pool", "check.cpp"), "-o", out])
    return out


@pytest.mark.parametrize("case", ["reuse", "handles", "captures", "many_calls", "all_in_use", "all_in_use_and_too_small"])
def test_blocks_wait_for_their_readers(check, case):
    cases = ["reuse", "handles", "captures", "many_calls", "all_in_use", "all_in_use_and_too_small"]
    r = subprocess.run([check, str(cases.index(case))], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
