"""Rounding errors of the membrane forces in the FP32 form: over the nodes of several meshes no larger (root mean
square, against the FP64 oracle) than those of the plain rules in correctly rounded FP32 arithmetic, which
plain_forces() evaluates on the CPU: positions, lengths squared and their differences to the relaxed values in FP64,
everything else in FP32, a node's edges, hinges and triangles added one after the other.  And meshes so small that
products of their lengths are FP32 denormals."""
import numpy as np
import pytest

import oracle as orc
from paper_1312_3426_amd import synth

from gpu_util import check, fmt, gpu_fields, oracle_fields, say

pytestmark = pytest.mark.gpu
f, d = np.float32, np.float64


def fma(a, b, c):
    return f(d(a) * d(b) + d(c))


def incidence(nv, owners, entries):
    """[k][nv]: the k-th entry of each node, -1 where it has fewer."""
    lists = [[] for _ in range(nv)]
    for v, e in zip(owners, entries):
        lists[v].append(e)
    out = np.full((max(len(x) for x in lists), nv), -1)
    for v, x in enumerate(lists):
        out[: len(x), v] = x
    return out


def plain_forces(R, x, ks=0.0, kb=0.0, kal=0.0, kag=0.0, kv=0.0, model="paper"):
    T, H, nv, cons = R.tris, R.hinges, R.nv, model != "paper"
    F = np.zeros((nv, 3), f)

    def add(owners, coef, vec):  # F_v += coef * vec, one entry of each node at a time
        nonlocal F
        for k in incidence(nv, owners, np.arange(len(owners))):
            c = np.where(k >= 0, coef[k], f(0))[:, None]
            F = fma(c, vec[k], F)

    a, b, c = (x[T[:, k]] for k in range(3))
    N = np.cross(b - a, c - a)
    n2 = (N * N).sum(1)
    ln = np.sqrt(f(n2))
    S = f(0.5) * ln
    dS = f(0.25 * n2 - R.S0 * R.S0) / (S + f(R.S0))
    normal = f(N) / ln[:, None]
    sg = d(dS).sum()
    vol = -((a - x[0]) * N).sum() / 6.0
    pa, pb, pc, pd = (x[H[:, k]] for k in range(4))
    e = pc - pb
    L2 = (e * e).sum(1)
    L = np.sqrt(L2)
    if ks:
        strain = f(L2 - R.L0 * R.L0) / (f(R.L0) * f(L + R.L0))
        lam = f(1) + strain
        sl, l2 = np.sqrt(lam), lam * lam
        s = f(ks) * ((sl + f(1) / (l2 * sl)) / (lam + f(1) / (l2 * lam))) * strain / f(L)
        add(np.concatenate([H[:, 1], H[:, 2]]), np.concatenate([s, s]), f(np.concatenate([e, -e])))
    if kb:
        n1, nn2 = np.cross(pb - pa, e), np.cross(e, pc - pd)
        md, dot = (np.cross(n1, nn2) * e).sum(1), (n1 * nn2).sum(1) * L
        c0, s0 = np.cos(R.theta0 - np.pi), np.sin(R.theta0 - np.pi)
        dth = f(np.arctan2(d(f(md * c0 - dot * s0)), d(f(dot * c0 + md * s0))))
        w = f(kb) * dth / f(R.theta0)
        if cons:
            c_ = f(R.hbar) * w
            wA, wD = (c_ * f(L) / f(np.sqrt((n * n).sum(1))) for n in (n1, nn2))
            aA, aD = f(((pa - pb) * e).sum(1) / L2), f(((pd - pb) * e).sum(1) / L2)
            roles = [(wA, 0), (-(f(1) - aA) * wA, -(f(1) - aD) * wD), (-aA * wA, -aD * wD), (0, wD)]
        else:
            roles = [(w, 0), (f(-0.5) * w, f(-0.5) * w), (f(-0.5) * w, f(-0.5) * w), (0, w)]
        t1, t2 = normal[R.hinge_tri[:, 0]], normal[R.hinge_tri[:, 1]]
        term = [fma((np.zeros_like(w) + p)[:, None], t1, (np.zeros_like(w) + q)[:, None] * t2) for p, q in roles]
        add(H.T.ravel(), np.ones(4 * len(H), f), np.concatenate(term))
    if kal or kag or kv:
        cg, cv = f(-kag * sg / (R.Sg0 + sg)), f(-kv * (vol - R.V0) / R.V0)
        g = (a + b + c) * (1.0 / 3.0)
        w = [f(p - g) for p in (a, b, c)]
        m2 = [(q * q).sum(1, dtype=f) for q in w]
        if cons:
            m2 = [(m2[0] + m2[1] + m2[2]) * f(1 / 3)] * 3
        vf = (cv * S * f(1 / 3))[:, None] * normal
        term = [fma((fma(-f(kal), dS / S, cg) / np.sqrt(q))[:, None], p, -vf) for p, q in zip(w, m2)]
        add(T.T.ravel(), np.ones(3 * len(T), f), np.concatenate(term))
    return d(F)


FAMILIES = {"stretching": dict(ks=0.05), "bending": dict(kb=0.02), "area": dict(kal=0.05, kag=0.2), "volume": dict(kv=0.3),
            "all": dict(ks=0.05, kb=0.02, kal=0.05, kag=0.2, kv=0.3)}


@pytest.mark.parametrize("model", ["paper", "conservative"])
@pytest.mark.parametrize("family", sorted(FAMILIES))
def test_error_of_the_forces(family, model):
    """From rest, without friction and with unit masses, one step leaves the force in the velocity."""
    from paper_1312_3426_amd import oif

    k = FAMILIES[family]
    gpu = plain = 0.0
    for seed in range(12):
        rng = np.random.default_rng(seed)
        n, t = (synth.icosphere(3, 4.0), synth.rbc_393(4.0))[seed % 2]
        n = n @ synth.random_rotation(rng).T
        edge = np.linalg.norm(n[t[:, 0]] - n[t[:, 1]], axis=1).mean()
        box = synth.Box(16, 16, 16, friction=0.0, templates=[synth.Template(n, t, model=model, **k)],
                        objects=[synth.ObjectSpec(0, np.array([8.0, 8.0, 8.0]))])
        x = n * (1.03 if seed < 8 else 0.95) + (0.001, 0.02, 0.15)[seed % 3] * edge * rng.standard_normal(n.shape)
        ctx = oif.Context.from_box(box, precision="fp32")
        ctx.write_mesh(-1, x + 8.0, np.zeros_like(x))
        x = ctx.read_mesh()[0] - 8.0  # as held
        ctx.step(1)
        v = ctx.read_mesh()[1]
        ctx.close()
        R = orc.Relaxed(n, t)
        ref = R.forces(x, model=model, **k)
        scale = np.sqrt((ref * ref).mean()) * 2.0 ** -24
        gpu += (((v - ref) / scale) ** 2).mean() / 12
        plain += (((plain_forces(R, x, model=model, **k) - ref) / scale) ** 2).mean() / 12
    say(f"[force error] {family} {model}: {np.sqrt(gpu):.3f} against {np.sqrt(plain):.3f} (2^-24 of the rms force)")
    assert np.isfinite(gpu) and gpu <= plain


@pytest.mark.parametrize("model", ["paper", "conservative"])
def test_mesh_whose_products_are_denormal(model):
    """Edges of some 2e-10: squared areas and the hinges' sines are products of four lengths, 1e-39 or so."""
    from paper_1312_3426_amd import oif

    say(f"[force error] denormal products {model}")
    n, t = synth.icosphere(2, 5e-10)
    box = synth.Box(16, 16, 16, friction=0.0, objects=[synth.ObjectSpec(0, np.zeros(3))],
                    templates=[synth.Template(n, t, kb=0.02, ks=0.01, kal=0.01, model=model)])
    ref = orc.System(box)
    ref.X[:] = n + 1.7e-12 * np.random.default_rng(0).standard_normal(n.shape)
    X0 = ref.X.copy()
    ctx = oif.Context.from_box(box, precision="fp32")
    ctx.write_mesh(-1, X0, np.zeros_like(X0))
    ctx.step(1)
    ref.run(1)
    res = check(gpu_fields(ctx, box.rho0, X0), oracle_fields(ref, X0), "fp32", box.rho0, 0.0, keys=("V",))
    ctx.close()
    say(fmt(res))
    assert all(v[3] for v in res.values()), fmt(res)
