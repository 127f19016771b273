"""Workgroups are dealt to the objects by their place, meshes of one size
together: whatever the number of each size (fewer than the 8 dies, a round of
them, one more, several rounds) and the order the objects were made in, every
object is stepped once.  Forces on the fluid are exact sums, so the results are
the same bits."""
import numpy as np
import pytest

from paper_1312_3426_amd import synth

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [(1, 1, 0), (3, 7, 2), (8, 8, 1), (9, 16, 0), (5, 17, 9)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_order_of_objects_does_not_show(prec, counts):
    from paper_1312_3426_amd import oif
    say(f"[order] {counts} objects {prec}")
    rng = np.random.default_rng(5)
    shapes = [synth.icosphere(1, 2.0), synth.icosphere(2, 3.0), synth.icosphere(3, 3.5)]
    kinds = np.repeat(np.arange(3), counts)
    specs = [(t, rng.uniform(-40, 80, 3)) for t in rng.permutation(kinds)]  # beyond the box as well
    out = []
    for perm in (np.arange(len(specs)), rng.permutation(len(specs))):
        box = synth.Box(48, 40, 36, templates=[synth.Template(n, t, ks=0.01, kb=1e-3) for n, t in shapes],
                        g=(1e-4, 0.0, 0.0), friction=0.1)
        box.objects = [synth.ObjectSpec(int(specs[k][0]), specs[k][1]) for k in perm]
        c = oif.Context.from_box(box, precision=prec)
        c.step(6)
        got = [None] * len(specs)
        for j, k in enumerate(perm):
            got[k] = c.read_mesh(j)
        out.append((c.read_velocity(), np.concatenate([np.stack(g, 1) for g in got])))
        assert np.isfinite(out[-1][1]).all() and np.abs(out[-1][1][:, 1]).min() > 0  # every node has moved
        c.close()
    assert (out[0][0] == out[1][0]).all() and (out[0][1] == out[1][1]).all()
