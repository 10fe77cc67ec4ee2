"""The host loops where the system refuses new threads (CPU, the library's own
host code): mmsd_set_m and mmsd_get_m run them for 262,144 nodes and more, and
an exception that leaves a C entry ends the caller's process."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1309_5796_amd", "csrc")


def test_loops_finish_without_new_threads(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "thread_start")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, os.path.join(ROOT, "tests", "native", "thread_start.cpp"),
                    os.path.join(CSRC, "amg.cpp"), "-o", exe, "-lpthread"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stderr)
    once, calls = map(int, re.findall(r"once (\d+) calls (\d+)", r.stdout)[0])
    assert once == 1 << 20 and calls == 1
