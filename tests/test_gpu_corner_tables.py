"""Meshes with nodes of many corners: latitude-longitude spheres, whose poles have one per meridian, whole in LDS and
split into patches; bipyramids in the global scratch, the larger one with a product of nodes and most corners (1.3e8)
beyond what 32-bit offsets of a rectangular table would reach.  Against the FP64 oracle with the criterion of gpu_util."""
import numpy as np
import pytest

from paper_1312_3426_amd import synth

from gpu_util import check, fmt, gpu_fields, oracle_fields, say

pytestmark = pytest.mark.gpu


def bipyramid(n):
    """n-gon with two apexes: n + 2 nodes, the apexes have n corners each."""
    phi = 2 * np.pi * np.arange(n) / n
    ring = np.stack([4 * np.cos(phi), 4 * np.sin(phi), np.zeros(n)], 1)
    nodes = np.concatenate([ring, [[0, 0, 3.0], [0, 0, -3.0]]])
    tris = [(k, (k + 1) % n, n + a) for k in range(n) for a in (0, 1)]
    return nodes, synth._orient_inward(nodes, np.array(tris, dtype=np.int32))


def globe(m, p):
    """Sphere of m meridians and p parallels: m p + 2 nodes, the poles have m corners each."""
    th = np.pi * np.arange(1, p + 1) / (p + 1)
    phi = 2 * np.pi * np.arange(m) / m
    ring = np.stack([np.outer(np.sin(th), np.cos(phi)), np.outer(np.sin(th), np.sin(phi)), np.outer(np.cos(th), np.ones(m))], 2)
    nodes = 4.0 * np.concatenate([ring.reshape(-1, 3), [[0, 0, 1.0], [0, 0, -1.0]]])
    tris = []
    for k in range(m):
        l = (k + 1) % m
        tris += [(k, l, m * p), (m * (p - 1) + k, m * (p - 1) + l, m * p + 1)]
        for j in range(p - 1):
            tris += [(m * j + k, m * j + l, m * j + m + k), (m * j + l, m * j + m + l, m * j + m + k)]
    return nodes, synth._orient_inward(nodes, np.array(tris, dtype=np.int32))


# (the bipyramids in the FP32 form alone: their wings are 8e-3 and 2e-3 high, where the positions' own rounding in the
# box shows in FP64)
CASES = [("globe_64x12", "fp32"), ("globe_64x12", "fp64"), ("globe_64x40", "fp32"), ("globe_64x40", "fp64"),
         ("bipyramid_3000", "fp32"), ("bipyramid_11600", "fp32")]


@pytest.mark.parametrize("model", ["paper", "conservative"])
@pytest.mark.parametrize("mesh,prec", CASES)
def test_nodes_of_many_corners_vs_oracle(mesh, prec, model):
    import oracle
    from paper_1312_3426_amd import oif

    say(f"[corner tables] {mesh} {prec} {model}")
    oracle.build()
    kind, size = mesh.split("_")
    nodes, tris = {"globe": globe, "bipyramid": bipyramid}[kind](*(int(v) for v in size.split("x")))
    tm = synth.Template(nodes, tris, ks=0.05, kb=0.02, kal=0.05, kag=0.2, kv=0.3, model=model)
    box = synth.Box(24, 20, 22, templates=[tm], objects=[synth.ObjectSpec(0, np.array([11.3, 9.8, 10.6]))])
    rng = np.random.default_rng(len(nodes))
    ref = oracle.System(box)
    edge = min(np.linalg.norm(nodes[t[k]] - nodes[t[k - 1]]) for t in tris for k in range(3))
    X0 = ref.X + 0.03 * edge * rng.standard_normal(ref.X.shape)
    V0 = 1e-3 * rng.standard_normal(ref.X.shape)
    ref.X[:], ref.V[:] = X0, V0
    ctx = oif.Context.from_box(box, precision=prec)
    ctx.write_mesh(-1, X0, V0)
    ctx.step(1)
    ref.run(1)
    res = check(gpu_fields(ctx, box.rho0, X0), oracle_fields(ref, X0), prec, box.rho0, 24)
    i = ctx.info()
    ctx.close()
    say(f"   LDS {i.lds_objects}, split {i.split_objects}, coupling in LDS {i.cpl_objects}: {fmt(res)}")
    if prec == "fp32":
        assert (i.lds_objects, i.split_objects) == {"globe_64x12": (1, 0), "globe_64x40": (0, 1)}.get(mesh, (0, 0))
    assert all(v[3] for v in res.values()), fmt(res)
