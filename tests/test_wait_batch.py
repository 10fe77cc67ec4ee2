"""The host's wait for a run (CPU, the library's own host code): it ends with the
outcome, with the batch, with an error, and with the run's time limit also
where the batch in flight never ends."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1309_5796_amd", "csrc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("wait") / "wait_batch")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, os.path.join(ROOT, "tests", "native", "wait_batch.cpp"),
                    "-o", out, "-lpthread"], check=True)
    return out


@pytest.mark.parametrize("what,end,polls", [("outcome", 0, 5), ("batch", 1, 7), ("hung", 2, 5000), ("late", 2, 0),
                                            ("error", 3, 3)])
def test_wait_ends(exe, what, end, polls):
    r = subprocess.run([exe, what], check=True, capture_output=True, text=True, timeout=30)
    assert tuple(map(int, re.findall(r"wait (\d) polls (\d+)", r.stdout)[0])) == (end, polls)
