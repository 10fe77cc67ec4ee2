"""The potential matrix without its zero couplings (CPU, the library's own
host code): on Kuhn boxes about half of the stored entries are exact zeros and
go, on jittered ones those of the air, on Delaunay meshes none; what remains
is symmetric, keeps every diagonal and gives the same product bit for bit."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from paper_1309_5796_amd import binding, meshgen

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1309_5796_amd", "csrc")

# mesh, and the range of the kept share of the entries
CASES = {
    "one_cell": (lambda: meshgen.kuhn_box((1e-9,) * 3, (1, 1, 1)), (0.4, 0.6)),
    "box": (lambda: meshgen.kuhn_box((5e-9, 6e-9, 3e-9), (5, 7, 3)), (0.4, 0.6)),
    "jittered": (lambda: meshgen.config1()["mesh"], (0.45, 0.7)),
    "delaunay": (lambda: meshgen.delaunay_box(3, n=9), (1.0, 1.0)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_zero_couplings_go_and_nothing_else(tmp_path, name):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "zero_couplings")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "zero_couplings.cpp"), os.path.join(CSRC, "amg.cpp"),
                    "-o", exe, "-lpthread"], check=True)
    make, (lo, hi) = CASES[name]
    a = binding.assembly_export(make())
    path = str(tmp_path / "L.bin")
    with open(path, "wb") as f:
        np.array([a["Nt"], len(a["lci"])], np.int32).tofile(f)
        a["lrp"].astype(np.int32).tofile(f)
        a["lci"].astype(np.int32).tofile(f)
        a["L"].astype(np.float64).tofile(f)
    out = subprocess.run([exe, path], check=True, capture_output=True, text=True).stdout
    n, nnz, kept, sym, ddev, dropped, same = re.findall(
        r"n (\d+) nnz (\d+) kept (\d+) sym (\d) ddev (\S+) dropped (\S+) same (\d)", out)[0]
    assert lo <= int(kept) / int(nnz) <= hi, out
    assert sym == "1" and same == "1" and float(ddev) == 0.0, out
    assert float(dropped) == 0.0, out   # the host assembly's zeros are exact
