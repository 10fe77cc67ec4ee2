"""The potential-matrix entries that bench.py's bytes model counts (CPU): those
the device holds, not the assembled ones."""
import numpy as np
import pytest

import bench
from paper_1309_5796_amd import binding, meshgen


@pytest.mark.parametrize("mesh,share", [(lambda: meshgen.kuhn_box((5e-9, 6e-9, 3e-9), (5, 7, 3)), (0.4, 0.6)),
                                        (lambda: meshgen.config1()["mesh"], (0.45, 0.7)),
                                        (lambda: meshgen.delaunay_box(3, n=9), (1.0, 1.0))])
def test_stored_entries(mesh, share):
    mesh = mesh()
    a = binding.assembly_export(mesh)
    n = bench.stored_potential_entries(mesh)
    # the host assembly's zero couplings are exact zeros
    assert n == np.count_nonzero(a["L"])
    assert share[0] <= n / len(a["L"]) <= share[1]


def test_sizes_carry_the_stored_entries():
    class P:
        def sizes(self):
            return dict(N=8, nnz_magnet=1, Nt=2, nnz_potential=99)

    cfg = dict(mesh=meshgen.delaunay_box(3, n=9))
    n = bench.stored_potential_entries(cfg["mesh"])
    assert bench.stored_sizes(P(), cfg) == dict(N=8, nnz_magnet=1, Nt=2, nnz_potential=n)
    cfg["stored_potential_entries"] = 5   # counted once per workload
    assert bench.stored_sizes(P(), cfg)["nnz_potential"] == 5
