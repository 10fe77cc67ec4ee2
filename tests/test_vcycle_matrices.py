"""The matrices of the device's V-cycle against the plain cycle's operations
(CPU, the library's own host code), on meshes of one to three levels."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from paper_1309_5796_amd import binding, meshgen

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1309_5796_amd", "csrc")

MESHES = {"config1": lambda: meshgen.config1()["mesh"], "box": lambda: meshgen.kuhn_box((7e-9, 9e-9, 5e-9), (7, 9, 5)),
          "ball": lambda: meshgen.kuhn_ball(cells=18), "delaunay": lambda: meshgen.delaunay_box(4, n=13)}


@pytest.mark.parametrize("name", sorted(MESHES))
def test_matrices_give_the_plain_cycle(tmp_path, name):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "vcycle_matrices")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, os.path.join(ROOT, "tests", "native", "vcycle_matrices.cpp"),
                    os.path.join(CSRC, "amg.cpp"), "-o", exe, "-lpthread"], check=True)
    a = binding.assembly_export(MESHES[name]())
    path = str(tmp_path / "L.bin")
    with open(path, "wb") as f:
        np.array([a["Nt"], len(a["lci"])], np.int32).tofile(f)
        a["lrp"].astype(np.int32).tofile(f)
        a["lci"].astype(np.int32).tofile(f)
        a["L"].astype(np.float64).tofile(f)
    out = subprocess.run([exe, path], check=True, capture_output=True, text=True).stdout
    rows = re.findall(r"post (\S+) fused (\S+) adj (\S+)", out)
    assert rows, out
    # sums of at most ~100 rounded products: 100 x 1.1e-16 and the same again
    # for the values of T, M and C themselves
    for post, fused, adj in rows:
        assert max(float(post), float(fused), float(adj)) < 1e-13, out
