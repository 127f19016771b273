"""The state sums at the sizes where their one launch changes shape: fewer
nodes than a block has threads, one node more or less than whole blocks, more
nodes than the most blocks take in one round, fewer and more membranes than
the last block has threads for; against FP64 sums of the same state read back,
twice with the same bits.  A sum of n terms in any order is off by at most
n * 2^-53 * sum |term| from the exact one."""
import math

import numpy as np
import pytest

import oracle as orc
from paper_1312_3426_amd import synth

from gpu_util import say

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("shape,cells", [((5, 3, 2), 0), ((11, 31, 3), 0), ((16, 8, 8), 0), ((25, 41, 1), 0),
                                         ((97, 83, 65), 3), ((40, 40, 40), 600)])
def test_sums_match_the_state(prec, shape, cells):
    from paper_1312_3426_amd import oif
    say(f"[diag] {shape} {cells} cells {prec}")
    rng = np.random.default_rng(3)
    n, t = synth.tetrahedron(0.8)
    box = synth.Box(*shape, templates=[synth.Template(n, t)], g=(0.0, 0.0, 0.0))
    box.objects = [synth.ObjectSpec(0, c) for c in 0.5 + rng.integers(0, shape, (cells, 3))]
    c = oif.Context.from_box(box, precision=prec)
    c.write_deviations(1e-3 * rng.standard_normal((19,) + shape[::-1]))
    if cells:
        X, _ = c.read_mesh()
        c.write_mesh(-1, X, 1e-3 * rng.standard_normal(X.shape))
    got = c.diagnostics()
    d = c.read_deviations()
    N = math.prod(shape)
    E = orc.D3Q19_E.astype(float)
    got4 = np.array([got.mass - N, *got.momentum_fluid])
    for k in range(4):
        term = (d if k == 0 else d * E[:, k - 1].reshape(19, 1, 1, 1)).ravel()
        # the mass is returned with N rho0 added, a sum rounded once
        bound = 19 * N * EPS * np.abs(term).sum() + (2 * EPS * N if k == 0 else 0)
        assert abs(got4[k] - math.fsum(term)) <= bound
    _, V = c.read_mesh()
    if prec != "fp64":  # what was written is read back as given; the device holds it in FP32
        V = V.astype(np.float32).astype(float)
    for k in range(3):
        assert abs(got.momentum_mesh[k] - math.fsum(V[:, k])) <= max(1, len(V)) * 2 * EPS * np.abs(V[:, k]).sum()
    again = c.diagnostics()
    assert (got.mass, *got.momentum_fluid, *got.momentum_mesh) == (again.mass, *again.momentum_fluid,
                                                                    *again.momentum_mesh)
    assert got.nonfinite == 0
    d = d.copy()
    d.flat[-1] = np.nan  # the last node of the last direction
    c.write_deviations(d)
    assert c.diagnostics().nonfinite == 1
    c.close()
