"""The admission estimate against the device memory that problem creation takes
through the context's allocator: meshes of one and two multigrid levels, whose
hierarchy is mostly the dense matrices of the coarsest level, and stretched
cells, which coarsen slowly."""
import numpy as np
import pytest

from paper_1309_5796_amd import meshgen

pytestmark = pytest.mark.gpu

MESHES = {
    "cube3": lambda: meshgen.kuhn_box((3e-9,) * 3, (3,) * 3),
    "cube10": lambda: meshgen.kuhn_box((10e-9,) * 3, (10,) * 3),
    "cube12": lambda: meshgen.kuhn_box((12e-9,) * 3, (12,) * 3),
    "cube15": lambda: meshgen.kuhn_box((15e-9,) * 3, (15,) * 3),
    "jittered11": lambda: meshgen.kuhn_box((11e-9,) * 3, (11,) * 3, jitter=0.1, rng=np.random.default_rng(2)),
    "jittered14": lambda: meshgen.kuhn_box((14e-9,) * 3, (14,) * 3, jitter=0.1, rng=np.random.default_rng(2)),
    "box16x16x8": lambda: meshgen.kuhn_box((12.8e-9, 12.8e-9, 6.4e-9), (16, 16, 8)),
    "box20x20x10": lambda: meshgen.kuhn_box((16e-9, 16e-9, 8e-9), (20, 20, 10)),
    "rod10": lambda: meshgen.kuhn_box((2e-9, 2e-9, 100e-9), (10, 10, 10)),
    "film12": lambda: meshgen.kuhn_box((50e-9, 50e-9, 1e-9), (24, 24, 12)),
    "delaunay17": lambda: meshgen.delaunay_box(6, n=17),
}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", sorted(MESHES))
def test_footprint_covers_one_and_two_level_hierarchies(name, precision):
    from paper_1309_5796_amd import binding
    print(f"[gpu] footprint {name} {precision}", flush=True)
    mesh, prec = MESHES[name](), binding.FP64 if precision == "fp64" else binding.MIXED
    ctx = binding.Context(0)
    p = binding.Problem(ctx, mesh, precision=prec)
    try:
        used = sum(t.numel() for t in ctx._alloc.live.values())
        est = binding.footprint(mesh, prec)
        print(f"  allocated {used / 1e6:.1f} MB, footprint {est / 1e6:.1f} MB", flush=True)
        assert 0 < used <= est
    finally:
        p.close()
        ctx.close()
