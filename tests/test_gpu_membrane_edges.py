"""GPU parity of the membrane kernel at the edges of its index lists and
workgroups: nodes with three to sixty-three corners (the first six are read
ahead, the others in a loop), meshes of 64 and 65 nodes, a node two closed
surfaces share, hinges bent past the range of the FP32 angle series; against
the FP64 oracle with the criterion of gpu_util, whole meshes in LDS."""
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


def two_tetrahedra():
    """Two tetrahedra with one common node (node 0)."""
    v, f = synth.tetrahedron(4.0)
    v = v - v[0]
    nodes = np.concatenate([v, -v[1:]])
    second = np.where(f == 0, 0, f + 3)
    return nodes, np.concatenate([f, second[:, [0, 2, 1]]]).astype(np.int32)


MESHES = {"tetrahedron": lambda: synth.tetrahedron(5.0), "octahedron": lambda: synth.octahedron(5.0),
          "two_tetrahedra": two_tetrahedra, "bipyramid_7": lambda: bipyramid(7),
          "bipyramid_62": lambda: bipyramid(62), "bipyramid_63": lambda: bipyramid(63)}


@pytest.mark.parametrize("model", ["paper", "conservative"])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("mesh", sorted(MESHES))
def test_odd_meshes_vs_oracle(mesh, prec, model):
    import oracle
    from paper_1312_3426_amd import oif

    say(f"[membrane edges] {mesh} {prec} {model}")
    oracle.build()
    nodes, tris = MESHES[mesh]()
    tm = synth.Template(nodes, tris, ks=0.05, kb=0.02, kal=0.05, kag=0.2, kv=0.3, model=model)
    box = synth.Box(24, 20, 22, templates=[tm], objects=[synth.ObjectSpec(0, np.array([11.3, 9.8, 10.6]))])
    rng = np.random.default_rng(len(nodes))
    ref = oracle.System(box)
    # displaced by 6 % of the shortest edge: bends hinges by some tenths, folds none
    edge = min(np.linalg.norm(nodes[t[k]] - nodes[t[k - 1]]) for t in tris for k in range(3))
    X0 = ref.X + 0.06 * edge * rng.standard_normal(ref.X.shape)
    V0 = 1e-3 * rng.standard_normal(ref.X.shape)
    ref.X[:], ref.V[:] = X0, V0
    ctx = oif.Context.from_box(box, precision=prec)
    ctx.write_mesh(-1, X0, V0)
    for block in (64, 256, 1024):
        ctx.set_launch(-1, block, -1)
        ctx.step(1)
        ref.run(1)
        res = check(gpu_fields(ctx, box.rho0, X0), oracle_fields(ref, X0), prec, box.rho0, 24)
        say(f"   {block} threads: {fmt(res)}")
        assert all(v[3] for v in res.values()), fmt(res)
    ctx.close()


@pytest.mark.parametrize("overlap", [False, True])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_runaway_mesh_takes_the_corner_path(prec, overlap):
    """A mesh spread over 2.4e6 lattice units per axis: the node count of its
    stencil box leaves 63 bits, and it must not pass for a small box.  Without
    moduli and friction the nodes fly straight and leave the fluid alone, so
    positions are exact and the fluid equals a box without cells."""
    from paper_1312_3426_amd import oif

    say(f"[membrane edges] runaway mesh {prec} overlap={overlap}")
    nodes, tris = synth.tetrahedron(5.0)
    box = synth.Box(24, 20, 22, templates=[synth.Template(nodes, tris)], friction=0.0,
                    objects=[synth.ObjectSpec(0, np.array([11.0, 9.0, 10.0]))])
    ctx = oif.Context.from_box(box, precision=prec)
    ctx.set_overlap(overlap)
    X0, _ = ctx.read_mesh()
    V = 1.2e6 * np.sign(nodes)  # extents of 2.4e6 after one step, 1.4e19 box nodes
    assert 2 ** 63 < int(2.4e6) ** 3 < 2 ** 64
    ctx.write_mesh(-1, X0, V)
    ctx.step(1)
    ctx.step(1)
    X, V1 = ctx.read_mesh()
    u = ctx.read_velocity()
    ctx.close()
    box.objects = []
    plain = oif.Context.from_box(box, precision=prec)
    plain.step(2)
    assert np.array_equal(V1, V) and np.array_equal(X, (X0 + V) + V)
    assert np.array_equal(u, plain.read_velocity())
    plain.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
def test_membrane_block_does_not_change_the_bits(prec):
    """The default workgroup size and set ones from one wave on (one, two and
    more waves fetch populations, or none), meshes in LDS and split ones: the
    same bits after five steps."""
    from paper_1312_3426_amd import oif

    say(f"[membrane edges] block sizes {prec}")
    box = synth.config_batch()[1]
    assert {o.tid for o in box.objects} == {0, 1, 2}
    got = []
    for block in (None, 64, 128, 192, 448, 768, 1024):
        c = oif.Context.from_box(box, precision=prec)
        rng = np.random.default_rng(3)
        X, _ = c.read_mesh()
        c.write_mesh(-1, X + 0.01 * rng.standard_normal(X.shape), 1e-3 * rng.standard_normal(X.shape))
        if block:
            c.set_launch(-1, block, -1)
        c.step(5)
        got.append((*c.read_mesh(), c.read_velocity()))
        c.close()
    for g in got[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(g, got[0]))
