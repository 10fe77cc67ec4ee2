"""Batches of both precisions at 8 and 16 lanes per magnet row, and with
different lanes for the two precisions (a launch per precision then), against
the same problems run one by one at the same block counts."""
import numpy as np
import pytest

from paper_1309_5796_amd import meshgen

pytestmark = pytest.mark.gpu

CELLS = (5, 8, 7)


@pytest.mark.parametrize("lanes_fp64,lanes_mixed", [(8, 8), (16, 16), (4, 16), (16, 8)])
def test_batch_matches_single_runs(lanes_fp64, lanes_mixed):
    from paper_1309_5796_amd import binding
    print(f"[gpu] batch lanes {lanes_fp64} {lanes_mixed}", flush=True)
    ctx = binding.Context(0)
    try:
        probs, single = [], []
        for k, n in enumerate(CELLS * 2):
            mixed = k >= len(CELLS)
            mesh = meshgen.kuhn_box((n * 1e-9,) * 3, (n,) * 3)
            p = binding.Problem(ctx, mesh, precision=binding.MIXED if mixed else binding.FP64)
            p.set_launch(lanes_mixed if mixed else lanes_fp64, 16)
            p.set_field(-1.0 * meshgen.U_H_1DEG)
            p.set_m(meshgen.noisy_plus_z(p.N, np.random.default_rng(n)))
            start = p.get_state()
            single.append((p.minimize(), p.get_m()))
            p.set_state(start)
            probs.append(p)
        out = binding.minimize_batch(probs)
        # the same decomposition and order of the sums: what may differ is the
        # compiler's contraction of products into sums, which reaches the end
        # as far as the stopping test lets it (the torque: 1e-6, FP32 fields)
        for k, (p, r) in enumerate(zip(probs, out)):
            ref, m = single[k]
            mixed = k >= len(CELLS)
            scale = abs(ref.e_exch_J) + abs(ref.e_anis_J) + abs(ref.e_zeem_J) + abs(ref.e_demag_J)
            assert r.status >= 0 and r.status == ref.status, k
            assert abs(r.energy_J - ref.energy_J) <= (1e-6 if mixed else 1e-10) * scale, k
            assert np.abs(p.get_m() - m).max() <= (1e-2 if mixed else 1e-5), k
        for p in probs:
            p.close()
    finally:
        ctx.close()
