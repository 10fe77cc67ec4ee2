"""Mixed-precision multigrid solves on odd-sized meshes in every V-cycle form, and
at a launch of few blocks, against the FP64 solution of the same state."""
import numpy as np
import pytest

from paper_1309_5796_amd import meshgen

pytestmark = pytest.mark.gpu

MESHES = {
    "cells5": lambda: meshgen.kuhn_box((5e-9, 5e-9, 5e-9), (5, 5, 5)),
    "flat": lambda: meshgen.kuhn_box((13e-9, 3e-9, 2e-9), (13, 3, 2)),
    "jittered11": lambda: meshgen.kuhn_box((11e-9,) * 3, (11,) * 3, jitter=0.1, rng=np.random.default_rng(2)),
    "cells16": lambda: meshgen.kuhn_box((16e-9,) * 3, (16,) * 3),   # finest level fused in this form only
    "ball21": lambda: meshgen.kuhn_ball(cells=21),
    "delaunay17": lambda: meshgen.delaunay_box(6, n=17),
}


@pytest.mark.parametrize("flags,blocks", [(None, 0), (0, 0), (4, 0), (7, 0), (3, 8)])
@pytest.mark.parametrize("name", sorted(MESHES))
def test_mixed_solve_matches_fp64(name, flags, blocks):
    from paper_1309_5796_amd import binding
    print(f"[gpu] mixed multigrid {name} flags={flags} blocks={blocks}", flush=True)
    mesh = MESHES[name]()
    ctx = binding.Context(0)
    if flags is not None:
        ctx.set_vcycle(flags)
    if blocks:
        ctx.set_launch_config(4, blocks)
    got = []
    try:
        for precision, rtol in ((binding.MIXED, 1e-6), (binding.FP64, 1e-12)):
            p = binding.Problem(ctx, mesh, precision=precision)
            m = meshgen.noisy_plus_z(p.N, np.random.default_rng(9), sigma=0.3)
            p.set_m(-m)
            p.evaluate()                      # another solve first: the checked one does not start from its answer
            p.set_m(m)
            r = p.evaluate(precond=binding.PRECOND_AMG, pcg_rtol=rtol)
            got.append((r, p.get_potential()))
            p.close()
    finally:
        ctx.close()
    (rm, um), (rd, ud) = got
    # a residual of 1e-6 |b| and the FP32 matrix: at most the condition number of
    # these matrices (below 1e4) times 1e-6, in the energy its square root
    assert 0 < rm.pcg_iters < 100 and 0 < rd.pcg_iters < 100
    assert np.linalg.norm(um - ud) <= 1e-2 * np.linalg.norm(ud)
    assert abs(rm.e_demag_J - rd.e_demag_J) <= 1e-4 * abs(rd.e_demag_J)
