"""The restriction that a fused level sweeps, against the residual it stands for
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

MESHES = {"cube3": lambda: meshgen.kuhn_box((3e-9,) * 3, (3,) * 3), "config1": lambda: meshgen.config1()["mesh"],
          "ball": lambda: meshgen.kuhn_ball(cells=18), "delaunay": lambda: meshgen.delaunay_box(4, n=13)}


@pytest.mark.parametrize("name", sorted(MESHES))
def test_restriction_of_the_residual(tmp_path, name):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "residual_restriction")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "residual_restriction.cpp"), os.path.join(CSRC, "amg.cpp"),
                    "-o", exe, "-lpthread"], check=True)
    a = binding.assembly_export(MESHES[name]())
    path = str(tmp_path / "L.bin")
    with open(path, "wb") as f:
        np.array([a["Nt"], len(a["lci"])], np.int32).tofile(f)
        a["lrp"].astype(np.int32).tofile(f)
        a["lci"].astype(np.int32).tofile(f)
        a["L"].astype(np.float64).tofile(f)
    out = subprocess.run([exe, path], check=True, capture_output=True, text=True).stdout
    devs = [float(d) for d in re.findall(r"dev (\S+)", out)]
    # sums of up to some hundred rounded products on either side
    assert devs and max(devs) < 1e-13, out
