"""Runs return while launches issued ahead are still queued on the stream.  What
a program does right after a run: change the launch shape or the material,
destroy the problem, run another problem of the context, restore a state; and
a run long enough for the host's looks at its progress, and one given up."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_1309_5796_amd import meshgen

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ctx():
    from paper_1309_5796_amd import binding
    c = binding.Context(0)
    yield c
    c.close()


def box(n, axis=(0.2, 0.1, 1.0), k1=meshgen.K1_JM3):
    mesh = meshgen.kuhn_box((n * 1e-9,) * 3, (n,) * 3)
    mesh.materials = [meshgen.Material(1, meshgen.JS_T, k1, meshgen.A_JM, np.array(axis))]
    return mesh


def problem(ctx, n, precision=0, **kw):
    from paper_1309_5796_amd import binding
    p = binding.Problem(ctx, box(n, **kw), precision=precision)
    p.set_field(-1.0 * meshgen.U_H_1DEG)
    p.set_m(meshgen.noisy_plus_z(p.N, np.random.default_rng(n)))
    return p


def scale(r):
    return abs(r.e_exch_J) + abs(r.e_anis_J) + abs(r.e_zeem_J) + abs(r.e_demag_J)


def bits(p, r):
    return r.status, r.energy_J, r.evals, r.pcg_iters, p.get_m().tobytes()


@pytest.mark.parametrize("precision", [0, 1])
def test_launch_shape_changed_right_after_a_run(ctx, precision):
    print(f"[gpu] run then set_launch precision={precision}", flush=True)
    p = problem(ctx, 7, precision)
    p.set_launch(4, 512)
    start = p.get_state()
    first = p.minimize(max_evals=8)
    p.set_launch(8, 64)
    m1 = p.get_m()
    p.set_state(start)
    other = p.minimize(max_evals=8)
    p.set_launch(4, 512)
    p.set_state(start)
    again = p.minimize(max_evals=8)
    # another order of the reductions: in FP64 rounding, and solves to 1e-10,
    # which eight steps carry along
    assert other.evals == 8 and np.isfinite(other.energy_J)
    assert precision or abs(other.energy_J - first.energy_J) <= 1e-8 * scale(first)
    assert (again.status, again.energy_J, again.evals, again.pcg_iters) == (first.status, first.energy_J, first.evals,
                                                                            first.pcg_iters)
    assert p.get_m().tobytes() == m1.tobytes()
    p.close()


def test_material_changed_right_after_a_run(ctx):
    print("[gpu] run then set_material", flush=True)
    p = problem(ctx, 6)
    p.evaluate()
    new = meshgen.Material(1, meshgen.JS_T, 0.5 * meshgen.K1_JM3, 0.7 * meshgen.A_JM, np.array([1.0, 0.3, 0.2]))
    p.set_material(new)
    got = p.evaluate()
    h = p.get_field()
    mesh = box(6)
    mesh.materials = [new]
    from paper_1309_5796_amd import binding
    q = binding.Problem(ctx, mesh)
    q.set_field(-1.0 * meshgen.U_H_1DEG)
    q.set_m(meshgen.noisy_plus_z(q.N, np.random.default_rng(6)))
    ref = q.evaluate(pcg_rtol=1e-12)
    # the stray field's solves stop at 1e-10 and 1e-12 of the right-hand side,
    # times a condition number of below 1e4; the other terms differ by rounding
    assert abs(got.energy_J - ref.energy_J) <= 1e-6 * scale(ref)
    assert abs(got.e_anis_J - ref.e_anis_J) <= 1e-12 * scale(ref)
    assert abs(got.e_exch_J - ref.e_exch_J) <= 1e-12 * scale(ref)
    assert np.abs(h - q.get_field()).max() <= 1e-6 * np.abs(h).max()
    p.close()
    q.close()


def test_problems_destroyed_right_after_their_runs(ctx):
    print("[gpu] run then destroy", flush=True)
    got = set()
    for _ in range(5):   # the next problem takes the memory of the last
        p = problem(ctx, 6)
        p.minimize(max_evals=6)
        p.close()
        p = problem(ctx, 6)
        r = p.evaluate()
        got.add((r.status, r.energy_J, r.pcg_iters, p.get_field().tobytes()))
        p.close()
    assert len(got) == 1


def test_problems_of_one_context_in_turn(ctx):
    print("[gpu] two problems in turn", flush=True)
    alone = []
    for n, prec in ((6, 0), (8, 1)):
        p = problem(ctx, n, prec)
        alone.append([bits(p, p.minimize(max_evals=k)) for k in (4, 3, 6)])
        p.close()
    a, b = problem(ctx, 6, 0), problem(ctx, 8, 1)
    for k, evals in enumerate((4, 3, 6)):
        ra, rb = a.minimize(max_evals=evals), b.minimize(max_evals=evals)   # nothing waits in between
        assert bits(a, ra) == alone[0][k] and bits(b, rb) == alone[1][k]
    a.close()
    b.close()


def test_a_run_of_many_batches(ctx, cfg1):
    """With every 32nd batch (after 744 launches, then 2,472) the host copies the
    control state to see that the run moves on."""
    from paper_1309_5796_amd import binding
    print("[gpu] run of many batches", flush=True)
    p = binding.Problem(ctx, cfg1["mesh"])
    p.set_field(cfg1["b_ext"])
    got = []
    for _ in range(2):
        p.set_m(cfg1["m0"])
        start = p.get_state()
        got.append(p.minimize(precond=binding.PRECOND_JACOBI))
        assert got[-1].status == 0 and got[-1].launches > 2600
        p.set_state(start)
    # the second run's first solve starts from another potential
    assert abs(got[0].energy_J - got[1].energy_J) <= 1e-10 * scale(got[0])
    p.close()


GIVEN_UP = """
import numpy as np
from paper_1309_5796_amd import binding, meshgen
ctx = binding.Context(0)
p = binding.Problem(ctx, meshgen.kuhn_box((6e-9,) * 3, (6,) * 3))
m = meshgen.noisy_plus_z(p.N, np.random.default_rng(1))
for _ in range(2):
    p.set_m(m)
    try:
        p.minimize()
    except Exception as e:
        print("given up:", e, flush=True)
    assert np.isfinite(p.get_m()).all()
p.close()
ctx.close()
print("closed", flush=True)
"""


def test_a_run_given_up_at_its_time_limit():
    """With a limit far below one batch's time: the run returns an error, and
    what follows on the problem is still ordered behind its launches."""
    print("[gpu] run given up", flush=True)
    r = subprocess.run([sys.executable, "-c", GIVEN_UP], cwd=ROOT, env=dict(os.environ, MMSD_RUN_TIMEOUT_S="1e-9"),
                       capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.count("given up: ") == 2 and r.stdout.count("MMSD_RUN_TIMEOUT_S") == 2
    assert r.stdout.rstrip().endswith("closed")
