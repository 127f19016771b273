"""Results on their way to the host in slots of half a MiB: node counts of one
slot, just over one, several, and so many that threads share them (32 MiB and
more), against what is known of the state: velocities against moments of the
populations read back, membranes without forces or friction against the
straight paths of their nodes; and several boxes read from threads at once."""
import threading

import numpy as np
import pytest

import oracle as orc
from paper_1312_3426_amd import synth

from gpu_util import say

pytestmark = pytest.mark.gpu
E64, E32 = 2.0 ** -53, 2.0 ** -24


def start(shape, prec, seed):
    from paper_1312_3426_amd import oif
    c = oif.Context.from_box(synth.Box(*shape, g=(1e-4, 2e-4, -1e-4)), precision=prec)
    c.write_deviations(1e-3 * np.random.default_rng(seed).standard_normal((19,) + shape[::-1]))
    return c


def check_fluid(c):
    d = c.read_deviations()
    rho, u = c.read_density(), c.read_velocity()
    E = orc.D3Q19_E.astype(float)
    size = np.abs(d).sum(axis=0)
    assert (np.abs(rho - 1.0 - d.sum(axis=0)) <= 40 * E64 * (1.0 + size)).all()
    for k, g in enumerate((1e-4, 2e-4, -1e-4)):
        j = np.tensordot(E[:, k], d, 1) + 0.5 * g
        assert (np.abs(u[k] - j / (1.0 + d.sum(axis=0))) <= 60 * E64 * (1.0 + size)).all()


@pytest.mark.parametrize("prec", ["fp64", "fp16"])
@pytest.mark.parametrize("shape", [(3, 5, 7), (43, 127, 4), (257, 17, 5), (131, 101, 107)])
def test_fields(prec, shape):  # 105, 21844, 21845 and 1415731 nodes; a slot holds 21845 velocities
    say(f"[read] {shape} {prec}")
    c = start(shape, prec, 1)
    check_fluid(c)
    c.close()


@pytest.mark.parametrize("prec,objects,integrator", [("fp64", 1, "euler"), ("fp32", 90, "euler"), ("fp32", 90, "verlet"),
                                                     ("fp32", 5800, "euler"), ("fp64", 4400, "verlet")])
def test_membranes(prec, objects, integrator):
    from paper_1312_3426_amd import oif
    say(f"[read] {objects} x 162 nodes {prec} {integrator}")
    rng = np.random.default_rng(2)
    n, t = synth.icosphere(2, 2.0)
    box = synth.Box(64, 64, 64, templates=[synth.Template(n, t)], g=(0.0, 0.0, 0.0), friction=0.0, integrator=integrator)
    box.objects = [synth.ObjectSpec(0, c) for c in rng.uniform(0, 64, (objects, 3))]
    c = oif.Context.from_box(box, precision=prec)
    X0, _ = c.read_mesh()
    V0 = 1e-2 * rng.standard_normal(X0.shape)
    c.write_mesh(-1, X0, V0)
    c.step(2)
    X, V = c.read_mesh()
    ev = E32 if prec != "fp64" else E64
    assert (np.abs(V - V0) <= 2 * ev * np.abs(V0)).all()
    assert (np.abs(X - X0 - 2 * V0) <= 8 * ev * np.abs(V0) + 16 * E64 * 64).all()
    k = objects - 1  # again, one membrane, from the host's copy
    Xk, Vk = c.read_mesh(k)
    assert (Xk == X[162 * k:]).all() and (Vk == V[162 * k:]).all()
    c.close()


def test_threads():
    say("[read] four boxes from four threads")
    boxes = [start((131, 101, 30 + k), "fp32", k) for k in range(4)]
    bad = []

    def read(c):
        try:
            for _ in range(3):
                check_fluid(c)
        except BaseException as e:
            bad.append(e)
    th = [threading.Thread(target=read, args=(c,)) for c in boxes]
    for x in th:
        x.start()
    for x in th:
        x.join()
    for c in boxes:
        c.close()
    assert not bad, bad
