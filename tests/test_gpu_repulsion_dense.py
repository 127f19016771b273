"""GPU parity of the pair search where cells hold several nodes: just under and over the node and a half a cell from
which the nodes are sorted by cell, and grids of five, three and two cells along an axis (the image by rounding);
periodic, between walls with nodes beyond them, and between walls that repel, cells in contact across faces of the box and drifting
across those of the grid, eager and captured steps; against the brute-force FP64 oracle with the criterion of gpu_util."""
import numpy as np
import pytest

from paper_1312_3426_amd import synth

from gpu_util import check, fmt, gpu_fields, oracle_fields, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("walls", ["periodic", "crossed", "repelling"])
@pytest.mark.parametrize("cutoff", [1.5, 2.0, 4.4, 7.3, 11.0])
def test_dense_pair_search_vs_oracle(cutoff, walls):
    import oracle
    from paper_1312_3426_amd import oif

    say(f"[repulsion dense] cutoff {cutoff} walls {walls}")
    oracle.build()
    nodes, tris = synth.icosphere(3, 2.5)
    box = synth.Box(24, 23, 22, walls_z=walls != "periodic", friction=0.2,
                    templates=[synth.Template(nodes, tris, ks=0.02, kv=0.1)],
                    repulsion=[synth.SoftSphere(0, 0, a=1e-6, n=2.0, cutoff=cutoff)])
    if walls == "repelling":
        box.repulsion.append(synth.SoftSphere(0, None, a=1e-5, n=1.2, cutoff=1.0))
    # two cells in contact across the x and y faces, one in the middle, one across or near the lower z face
    for o in ((0.4, 22.6, 11.0), (5.5, 22.8, 11.1), (12.0, 12.0, 11.0), (12.5, 13.0, 3.3 if walls == "repelling" else 2.1)):
        box.objects.append(synth.ObjectSpec(0, np.array(o)))
    rng = np.random.default_rng(6)
    ref = oracle.System(box)
    X0, V0 = ref.X + 0.01 * rng.standard_normal(ref.X.shape), 0.02 * rng.standard_normal(ref.X.shape)
    V0 += np.repeat([[-0.2, 0.15, 0.3], [-0.25, 0.15, -0.2], [0.4, -0.3, 0.1], [0.1, 0.1, -0.1]], len(nodes), 0)
    ref.X[:], ref.V[:] = X0, V0
    ctx = oif.Context.from_box(box, precision="fp64")
    ctx.write_mesh(-1, X0, V0)
    for n in (1, 4):
        ctx.set_graph(0 if n == 1 else 2)
        ctx.step(n)
        ref.run(n)
        res = check(gpu_fields(ctx, box.rho0, X0), oracle_fields(ref, X0), "fp64", box.rho0, 24)
        say(f"   after {n} more: {fmt(res)}")
        assert all(v[3] for v in res.values()), fmt(res)
    ctx.close()
