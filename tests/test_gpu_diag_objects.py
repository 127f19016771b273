"""State sums over many membranes, where objects share the blocks of the launch: one more than have a block each, a
last block that is not full, nodes at the limits of one and of four waves an object, unequal masses; against FP64 sums
of the velocities as the device holds them.  A sum of n terms in any order is off by at most n * 2^-53 * sum |term|."""
import math

import numpy as np
import pytest

from paper_1312_3426_amd import synth

from gpu_util import say

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


def prism(n):
    """Closed band of n - 2 sides with two poles: n nodes."""
    m = n - 2
    phi = 2 * np.pi * np.arange(m) / m
    nodes = np.concatenate([np.stack([np.cos(phi), np.sin(phi), 0 * phi], 1), [[0, 0, 1.0], [0, 0, -1.0]]])
    tris = [(k, (k + 1) % m, m + a) for k in range(m) for a in (0, 1)]
    return nodes, synth._orient_inward(nodes, np.array(tris, dtype=np.int32))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("count", [512, 513, 529, 1040])
@pytest.mark.parametrize("largest", [63, 64, 65, 256, 257, 1024, 1025])
def test_momentum_of_many_membranes(largest, count, prec):
    from paper_1312_3426_amd import oif
    say(f"[diag objects] {count} objects of up to {largest} nodes {prec}")
    rng = np.random.default_rng(largest)
    masses = (1.0, 2.5)
    tm = [synth.Template(*prism(n)) for n in (largest, 5)]
    box = synth.Box(24, 20, 16, templates=tm, g=(0.0, 0.0, 0.0))
    box.objects = [synth.ObjectSpec(int(k % 7 > 2), c, mass=masses[k % 2]) for k, c in enumerate(rng.uniform(0, 16, (count, 3)))]
    c = oif.Context.from_box(box, precision=prec)
    X, _ = c.read_mesh()
    V = 1e-3 * rng.standard_normal(X.shape)
    c.write_mesh(-1, X, V)
    d = c.diagnostics()
    if prec != "fp64":
        V = V.astype(np.float32).astype(float)
    m = np.concatenate([np.full(len(tm[o.tid].nodes), o.mass) for o in box.objects])
    for k in range(3):
        term = m * V[:, k]
        assert abs(d.momentum_mesh[k] - math.fsum(term)) <= len(term) * 2 * EPS * np.abs(term).sum()
    assert d.nonfinite == 0
    assert tuple(c.diagnostics_noalloc().momentum_mesh) == tuple(d.momentum_mesh)
    V[-1] = 1e308  # the last node of the last object: its components' sum is infinite
    c.write_mesh(-1, X, V)
    assert c.diagnostics().nonfinite == 1
    c.close()
