"""The slices' offsets near their 32-bit limit (CPU, the library's own host
code): matrices of 2^29 entries and more, which the multigrid levels of meshes
of some 50 million nodes have, fit; what needs more than 32 bits is refused."""
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
    out = str(tmp_path_factory.mktemp("slices") / "slice_offsets")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, os.path.join(ROOT, "tests", "native", "slice_offsets.cpp"),
                    os.path.join(CSRC, "amg.cpp"), "-o", out, "-lpthread"], check=True)
    return out


# rows, entries per row, entries of the first row, lanes per row, the last offset (None: refused)
@pytest.mark.parametrize("rows,length,first,lanes,last", [
    (1024, 1 << 19, 1 << 19, 1, 1 << 29), (1024, 1 << 20, 1 << 20, 1, 1 << 30), (1024, 2_000_000, 2_000_000, 32, 2_048_000_000),
    (64, 1, 33_554_431, 1, 64 * 33_554_431), (64, 1, 33_554_432, 1, None), (65, 1, 40_000_000, 1, None),
    (17, 3, 3, 4, 128), (1, 0, 0, 8, 0)])
def test_offsets(exe, rows, length, first, lanes, last):
    out = subprocess.run([exe, *map(str, (rows, length, first, lanes))], check=True, capture_output=True, text=True).stdout
    n, end = map(int, re.findall(r"offsets (\d+) last (-?\d+)", out)[0])
    per = 64 // lanes
    assert (n, end) == ((0, -1) if last is None else ((rows + per - 1) // per + 1, last))
