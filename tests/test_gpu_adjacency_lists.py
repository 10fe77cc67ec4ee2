"""Device assembly around a node whose adjacency list is shorter than, as long
as and longer than a wavefront, against the host assembly: bipyramids of k
slices, whose centre lies in 2 k tets."""
import numpy as np
import pytest

from paper_1309_5796_amd import meshgen

pytestmark = pytest.mark.gpu


def bipyramid(k):
    t = 2 * np.pi * np.arange(k) / k
    ring = np.stack([np.cos(t), np.sin(t), 0.05 * np.cos(3 * t)], axis=1)
    xyz = np.concatenate([[[0, 0, 0], [0.1, 0, 1], [0, 0.1, -1]], ring]) * 5e-9
    a, b = 3 + np.arange(k), 3 + (np.arange(k) + 1) % k
    o = np.zeros(k, int)
    tets = np.concatenate([np.stack([o, o + 1, a, b], axis=1), np.stack([o, o + 2, b, a], axis=1)]).astype(np.int32)
    tets = tets[np.random.default_rng(k).permutation(len(tets))]
    return meshgen.Mesh(xyz=xyz, tets=tets, region=np.ones(len(tets), np.int32),
                        dirichlet=np.zeros(len(xyz), np.uint8),
                        materials=[meshgen.Material(1, meshgen.JS_T, meshgen.K1_JM3, meshgen.A_JM, np.array([0.2, 0.1, 1.0]))])


@pytest.mark.parametrize("k", [5, 31, 32, 33, 70])
def test_assembly_around_a_node_in_2k_tets(k):
    from paper_1309_5796_amd import binding
    print(f"[gpu] adjacency lists k={k}", flush=True)
    mesh = bipyramid(k)
    host = binding.assembly_export(mesh)
    ctx = binding.Context(0)
    try:
        dev = {n: v.cpu().numpy() if hasattr(v, "cpu") else v for n, v in binding.assemble_device(ctx, mesh).items()}
    finally:
        ctx.close()
    for n in ("mrp", "mci"):
        assert np.array_equal(dev[n], host[n]), n
    # the same terms in the same order; the fused multiply-adds of the
    # geometry differ by rounding, once per incident tet
    for n in ("K", "D1", "D2", "Q", "V"):
        assert np.abs(dev[n] - host[n]).max() <= 1e-14 * max(1.0, 2 * k / 100) * np.abs(host[n]).max(), n
