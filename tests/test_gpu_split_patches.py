"""Split meshes with more patches in one launch than the device holds at once: a patch that starts after a neighbour
has ended stages the neighbour's nodes at the step's start all the same.  The same boxes stepped one by one, where all
patches run together, give the same bits."""
import numpy as np
import pytest

from paper_1312_3426_amd import synth

from gpu_util import say

pytestmark = pytest.mark.gpu


def boxes(n_boxes, per_box, integrator):
    n, t = synth.icosphere(4, 4.0)
    fine = {k: v * synth.FINE_MODULI_SCALE for k, v in synth.MODULI_DEFAULT.items()}
    out = []
    for b in range(n_boxes):
        at = np.random.default_rng(b).uniform(0, 40, (per_box, 3))
        out.append(synth.Box(40, 40, 40, g=(1e-5, 0.0, 0.0), friction=synth.WORKING_FRICTION_FINE, integrator=integrator,
                             templates=[synth.Template(n, t, **fine)], objects=[synth.ObjectSpec(0, x) for x in at]))
    return out


def start(box, prec, seed):
    from paper_1312_3426_amd import oif
    c = oif.Context.from_box(box, precision=prec)
    rng = np.random.default_rng(seed)
    X, _ = c.read_mesh()
    c.write_mesh(-1, X + 0.005 * rng.standard_normal(X.shape), 1e-3 * rng.standard_normal(X.shape))
    return c


@pytest.mark.parametrize("integrator", ["euler", "verlet"])
@pytest.mark.parametrize("prec,n_boxes", [("fp64", 10), ("fp32", 24)])
def test_more_patches_than_run_at_once(prec, n_boxes, integrator):
    from paper_1312_3426_amd import oif
    say(f"[split patches] {n_boxes} boxes of 12 spheres {prec} {integrator}")
    bx = boxes(n_boxes, 12, integrator)
    alone = []
    for k, b in enumerate(bx):
        c = start(b, prec, k)
        c.step(5)
        i = c.info()
        assert i.split_objects == 12 and i.split_workgroups == 48
        alone.append((*c.read_mesh(), c.read_velocity()))
        c.close()
    ctxs = [start(b, prec, k) for k, b in enumerate(bx)]
    batch = oif.Batch(ctxs)
    batch.step(5)
    for c, ref in zip(ctxs, alone):
        assert all(np.array_equal(a, r) for a, r in zip((*c.read_mesh(), c.read_velocity()), ref))
    batch.close()
    for c in ctxs:
        c.close()
