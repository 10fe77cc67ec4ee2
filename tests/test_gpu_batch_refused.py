"""A batch that is refused after its first table was uploaded (problems of one
precision with different lanes per row): the error, and the same problems run
correctly afterwards."""
import numpy as np
import pytest

from paper_1309_5796_amd import meshgen

pytestmark = pytest.mark.gpu


def test_refused_batch_leaves_the_problems_usable():
    from paper_1309_5796_amd import binding
    print("[gpu] refused batch", flush=True)
    ctx = binding.Context(0)
    try:
        probs, single = [], []
        for k, prec in enumerate((binding.FP64, binding.FP64, binding.MIXED, binding.MIXED)):
            p = binding.Problem(ctx, meshgen.kuhn_box((5e-9,) * 3, (5,) * 3), precision=prec)
            p.set_launch(4, 16)
            p.set_field(-1.0 * meshgen.U_H_1DEG)
            p.set_m(meshgen.noisy_plus_z(p.N, np.random.default_rng(k)))
            start = p.get_state()
            r = p.minimize(max_evals=6)
            single.append((r.energy_J, r.evals, p.get_m()))
            p.set_state(start)
            probs.append(p)
        probs[3].set_launch(8, 16)   # the FP64 table is on its way when the mixed one is refused
        for _ in range(3):
            with pytest.raises(Exception, match="lanes per row"):
                binding.minimize_batch(probs, max_evals=6)
        probs[3].set_launch(4, 16)
        out = binding.minimize_batch(probs, max_evals=6)
        for k, (p, r) in enumerate(zip(probs, out)):
            e, evals, m = single[k]
            assert r.evals == evals
            assert abs(r.energy_J - e) <= (1e-5 if k > 1 else 1e-10) * abs(e)
            assert np.abs(p.get_m() - m).max() <= (1e-3 if k > 1 else 1e-8)
        for p in probs:
            p.close()
    finally:
        ctx.close()
