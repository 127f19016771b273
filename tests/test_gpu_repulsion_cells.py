"""GPU parity of the pair search at the edges of its cell grid: ranges small
against the cells (two cells along an axis), between half a cell and a cell
(three), a grid of four and of two cells along an axis (the image by rounding),
periodic and between walls, cells drifting across faces of the box and of the
grid; against the brute-force FP64 oracle with the criterion of gpu_util."""
import numpy as np
import pytest

from paper_1312_3426_amd import synth

from gpu_util import check, fmt, gpu_fields, oracle_fields, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("cutoff", [0.3, 0.8, 5.9, 11.0])
def test_pair_search_vs_oracle(cutoff, walls):
    import oracle
    from paper_1312_3426_amd import oif

    say(f"[repulsion cells] cutoff {cutoff} walls {walls}")
    oracle.build()
    nodes, tris = synth.icosphere(2, 2.5)
    box = synth.Box(24, 23, 22, walls_z=walls, friction=0.2,
                    templates=[synth.Template(nodes, tris, ks=0.02, kv=0.1)],
                    repulsion=[synth.SoftSphere(0, 0, a=1e-5, n=2.0, cutoff=cutoff)])
    # two cells in contact across the x and y faces, one in the middle
    for o in ((0.4, 22.6, 11.0), (5.5, 22.8, 11.1), (12.0, 12.0, 11.0)):
        box.objects.append(synth.ObjectSpec(0, np.array(o)))
    rng = np.random.default_rng(5)
    ref = oracle.System(box)
    X0, V0 = ref.X + 0.01 * rng.standard_normal(ref.X.shape), 0.02 * rng.standard_normal(ref.X.shape)
    V0 += np.repeat([[-0.2, 0.15, 0.3], [-0.25, 0.15, -0.2], [0.4, -0.3, 0.1]], len(nodes), 0)
    ref.X[:], ref.V[:] = X0, V0
    ctx = oif.Context.from_box(box, precision="fp64")
    ctx.write_mesh(-1, X0, V0)
    for n in (1, 4):
        ctx.step(n)
        ref.run(n)
        res = check(gpu_fields(ctx, box.rho0, X0), oracle_fields(ref, X0), "fp64", box.rho0, 24)
        say(f"   after {n} more: {fmt(res)}")
        assert all(v[3] for v in res.values()), fmt(res)
    ctx.close()
