"""Timed cases of the coupled lattice-Boltzmann / membrane step, as a program of this library runs it: build a
box (or a batch of boxes), step it, read the meshes and the fluid velocity back.

A case is a dict of plain values:
  kind       "box" (one Context), "batch" (many boxes through Batch) or "observe" (short runs with a time series of
             diagnostics and cell analyses between them)
  nx, ny, nz box size; walls: bounce-back walls at both z ends; channel: the S-shaped obstacle channel with its inlet
  mesh       "ico2" / "ico3" / "ico4" (icospheres of 162 / 642 / 2562 nodes), "rbc393", "rbc642" (biconcave cells);
             radius: its radius; cells: how many
  prec       "fp64", "fp32", "fp16", "bf16" (storage form; the last two compute in FP32)
  steps      coupled steps of one pass; graph: steps per captured graph (0: eager launches); tune: autotuned launches
  mrt, verlet, repulsion, conservative: the engine's options
  batch      boxes: how many; mix: seed of the boxes' sizes and cells (the shapes belong to the case, not to its seed)
Cells sit at random sites of a grid that keeps them a lattice unit apart (with repulsion a fifth of one, within its
range), randomly turned, their nodes displaced and moving a little; small boxes start from a seeded flow, large ones
from rest."""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1312_3426_amd import oif, synth

MODULI = dict(synth.MODULI_DEFAULT)
FINE = {k: v * synth.FINE_MODULI_SCALE for k, v in MODULI.items()}  # the 2562-node sphere is stiffer (see synth)
MRT = (0.0, -0.5, 0.3, -0.3)
# Weaker than the 1e-5 of the short benchmark runs: a periodic box keeps accelerating, and a long series of passes on
# one state has to stay at low Mach numbers.
BODY_FORCE = (1e-6, 0.0, 0.0)
SOFT = synth.SoftSphere(0, 0, a=1e-7, n=2.0, cutoff=0.3)
NODES = {"ico2": 162, "ico3": 642, "ico4": 2562, "rbc393": 393, "rbc642": 642}
FLOW_NODES = 1 << 18  # boxes up to this size start from a seeded flow


def _box_case(name, nx, ny, nz, mesh, cells, prec, steps, **kw):
    c = dict(name=name, kind="box", nx=nx, ny=ny, nz=nz, mesh=mesh, radius=4.0, cells=cells, prec=prec, steps=steps,
             graph=0, tune=False, walls=False, channel=False, mrt=False, verlet=False, repulsion=False,
             conservative=False)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one step of the FP64 method case (one sphere in 20^3), fields read after it, as a program
        # does that couples the step to something else
        _box_case("sphere_20_fp64_1step", 20, 20, 20, "ico3", 1, "fp64", 1),
        # the channel case: ten red cells between walls, short graph runs
        _box_case("channel_64_fp32", 64, 32, 32, "rbc393", 10, "fp32", 100, graph=50, walls=True),
        # the headline workload in its FP32 and FP16 forms, as the benchmark runs it (autotuned, graphs of 50 steps)
        _box_case("spheres_256_fp32", 256, 128, 128, "ico3", 500, "fp32", 500, graph=50, tune=True),
        _box_case("spheres_256_fp16", 256, 128, 128, "ico3", 500, "fp16", 500, graph=50, tune=True),
        # odd sizes that fill no tile, BF16 storage, the engine's own collision and integrator, eager launches
        _box_case("ragged_bf16_mrt_verlet", 191, 101, 77, "rbc393", 150, "bf16", 300, mrt=True, verlet=True),
        # suspension with cell-cell repulsion, MRT and Verlet (the engine's options together)
        _box_case("repulsion_256_fp32", 256, 128, 128, "ico3", 500, "fp32", 300, graph=50, mrt=True, verlet=True,
                  repulsion=True),
        # the S-shaped obstacle channel with moving inlet
        _box_case("obstacles_384_fp32", 384, 192, 64, "rbc393", 400, "fp32", 300, graph=50, walls=True, channel=True),
        # the largest: 5000 cells of diameter 15; a program that follows the cells reads the meshes, not the field
        _box_case("scale_512_fp32", 512, 256, 256, "rbc642", 5000, "fp32", 200, graph=50, tune=True, radius=7.5),
        # FP64 form with the conservative force model, eager launches
        _box_case("conservative_128_fp64", 128, 128, 128, "ico3", 120, "fp64", 100, conservative=True),
        # 32 uneven boxes with 1 to 20 cells of 162 to 2562 nodes each, stepped as one batch
        dict(name="batch_32_fp32", kind="batch", boxes=32, mix=4, prec="fp32", steps=200, graph=50),
        # time series: short runs, each followed by diagnostics, the meshes and one analysis per cell
        _box_case("observe_128_fp32", 128, 64, 64, "rbc393", 40, "fp32", 100, kind="observe"),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed ones' ranges: sizes by logarithm, odd ones among them, any form and option."""
    kind = rng.choice(["box", "box", "box", "box", "batch", "observe"])
    prec = rng.choice(["fp64", "fp32", "fp32", "fp16", "bf16"])
    graph = rng.choice([0, 50])
    if kind == "batch":
        return dict(kind="batch", boxes=_logint(rng, 2, 32), mix=rng.randrange(1 << 20), prec=prec,
                    steps=_logint(rng, 50, 200), graph=graph)
    channel = kind == "box" and rng.random() < 0.2
    verlet = rng.random() < 0.3
    mesh = rng.choice(["ico2", "ico3", "rbc393", "rbc642"])
    radius = 7.5 if mesh == "rbc642" else 4.0
    nx, ny, nz = _logint(rng, 24, 320), _logint(rng, 20, 160), _logint(rng, 20, 128)
    if channel:
        nx, ny, nz = _logint(rng, 96, 384), _logint(rng, 64, 192), _logint(rng, 24, 64)
        mesh, radius = "rbc393", 4.0
    walls = channel or rng.random() < 0.3
    nx, ny, nz = (max(v, int(2 * radius) + 12) for v in (nx, ny, nz))
    c = _box_case("", nx, ny, nz, mesh, 0, prec, 0, graph=graph, radius=radius, walls=walls, channel=channel,
                  mrt=rng.random() < 0.3, verlet=verlet, repulsion=rng.random() < 0.2,
                  conservative=rng.random() < 0.2, kind=kind)
    del c["name"]
    c["cells"] = max(1, int(len(_sites(c)) * rng.uniform(0.03, 0.3)))
    n = nx * ny * nz
    c["steps"] = 100 if kind == "observe" else max(1, min(300, int(2e9 / n)) - rng.randrange(3))
    return c


# ---- inputs -------------------------------------------------------------------------------------------------------


def _room(case):
    """Gap of the placement grid's cells and the jitter of their centres. Closer cells without repulsion let their
    nodes share lattice nodes, where the explicit drag of the finest mesh is no longer stable."""
    return (1.0, 0.4) if case["repulsion"] else (1.4, 0.2)


def _sites(case):
    """Cell centres a box has room for: a regular grid, clear of the walls and of the channel's obstacles."""
    r, room = case["radius"], _room(case)[0]
    dims = (case["nx"], case["ny"], case["nz"])
    lo, hi = [0.0] * 3, [float(d) for d in dims]
    if case["walls"]:
        lo[2], hi[2] = r + 1.5, dims[2] - r - 1.5
    axes = []
    for a in range(3):
        wall = a == 2 and case["walls"]
        n = int((hi[a] - lo[a]) / (2 * r + room)) + (1 if wall else 0)
        n = max(1, n)
        h = (hi[a] - lo[a]) / (max(1, n - 1) if wall else n)
        axes.append(lo[a] + h * (np.arange(n) + (0.0 if wall and n > 1 else 0.5)))
    s = np.stack(np.meshgrid(*axes, indexing="ij"), axis=-1).reshape(-1, 3)
    if case["channel"]:
        nx, ny = dims[:2]
        keep = (s[:, 1] > 2 + r + 1.5) & (s[:, 1] < ny - 2 - r - 1.5) & (s[:, 0] > 2 + r + 1.5) & (s[:, 0] < nx - r - 1.5)
        for b in synth.obstacle_channel_boundaries(nx, ny)[2:4]:
            x0, y0 = b.corner[:2]
            keep &= ~((s[:, 0] > x0 - r - 1.5) & (s[:, 0] < x0 + b.a[0] + r + 1.5) &
                      (s[:, 1] > y0 - r - 1.5) & (s[:, 1] < y0 + b.b[1] + r + 1.5))
        s = s[keep]
    return s


_MESH = {}


def _mesh(name, radius):
    if (name, radius) not in _MESH:
        _MESH[name, radius] = (synth.icosphere(int(name[3:]), radius) if name.startswith("ico") else
                               synth.rbc_393(radius) if name == "rbc393" else synth.rbc_642(radius))
    return _MESH[name, radius]


def _template(mesh, radius, conservative):
    return synth.Template(*_mesh(mesh, radius), **(FINE if mesh == "ico4" else MODULI),
                          model="conservative" if conservative else "paper")


def _place(rng, case, meshes):
    """The cells at random sites: `meshes[k]` is the template of cell k."""
    s = _sites(case)
    jitter = _room(case)[1]
    at = s[rng.choice(len(s), size=len(meshes), replace=False)] + rng.uniform(-jitter, jitter, (len(meshes), 3))
    return [synth.ObjectSpec(t, x, synth.random_rotation(rng)) for t, x in zip(meshes, at)]


def _boxes(case, seed):
    rng = np.random.default_rng(seed)
    if case["kind"] != "batch":
        nx, ny, nz = case["nx"], case["ny"], case["nz"]
        objs = _place(rng, case, [0] * case["cells"])
        return [synth.Box(nx, ny, nz, g=(0.0, 0.0, 0.0) if case["channel"] else BODY_FORCE, walls_z=case["walls"],
                          templates=[_template(case["mesh"], case["radius"], case["conservative"])], objects=objs,
                          boundaries=synth.obstacle_channel_boundaries(nx, ny) if case["channel"] else [],
                          mrt=MRT if case["mrt"] else None, integrator="verlet" if case["verlet"] else "euler",
                          repulsion=[SOFT] if case["repulsion"] else [])], rng
    shape = np.random.default_rng(case["mix"])
    tmpl = [_template(m, 4.0, False) for m in ("ico2", "ico3", "ico4")]
    out = []
    for b in range(case["boxes"]):
        dims = (int(shape.integers(32, 65)), int(shape.integers(32, 49)), int(shape.integers(32, 49)))
        levels = [int(v) for v in shape.integers(0, 3, size=int(shape.integers(1, 21)))]
        c = dict(nx=dims[0], ny=dims[1], nz=dims[2], radius=4.0, walls=False, channel=False, repulsion=False)
        out.append(synth.Box(*dims, g=BODY_FORCE, friction=synth.WORKING_FRICTION_FINE, templates=tmpl,
                             objects=_place(rng, c, levels)))
    return out, rng


def _start(box, rng):
    """Mesh displacement and velocity (per node), and the starting deviations of a small box (None: rest)."""
    m = box.n_mesh_nodes
    dx = 0.01 * rng.standard_normal((m, 3))
    v = 1e-4 * rng.standard_normal((m, 3))
    if box.n_nodes > FLOW_NODES or box.boundaries:
        return dx, v, None
    x, y, z = (2 * math.pi * (np.arange(n) + 0.5) / n for n in (box.nx, box.ny, box.nz))
    ph = rng.uniform(0, 2 * math.pi, 3)
    u = np.zeros((3, box.nz, box.ny, box.nx))  # a shear wave per axis pair
    u[0] += 2e-3 * np.sin(y + ph[0])[None, :, None]
    u[1] += 2e-3 * np.sin(z + ph[1])[:, None, None]
    u[2] += 2e-3 * np.sin(x + ph[2])[None, None, :] * (0.0 if box.walls_z else 1.0)
    usq = 1.5 * (u * u).sum(0)
    d = np.empty((19, box.nz, box.ny, box.nx))
    for i in range(19):
        eu = sum(E[i][a] * u[a] for a in range(3))
        d[i] = W[i] * (3 * eu + 4.5 * eu * eu - usq)
    return dx, v, d


def prepare(case, seed):
    boxes, rng = _boxes(case, seed)
    ctxs = []
    for b in boxes:
        c = oif.Context.from_box(b, precision=case["prec"])
        dx, v, d = _start(b, rng)
        x0, _ = c.read_mesh()
        c.write_mesh(-1, x0 + dx, v)
        if d is not None:
            c.write_deviations(d)
        if case.get("tune"):
            c.autotune()
        ctxs.append(c)
    batch = oif.Batch(ctxs) if case["kind"] == "batch" else None
    if case["graph"]:
        (batch or ctxs[0]).set_graph(case["graph"])
    return dict(case=case, ctxs=ctxs, batch=batch)


# ---- one pass -----------------------------------------------------------------------------------------------------

# The library hands every form's fields over in FP64; a program keeps them in the form's own type.
KEEP = {"fp64": torch.float64, "fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}


def _keep(case, a):
    return torch.from_numpy(a).to(KEEP[case["prec"]])


def _reads_velocity(case):
    return case["kind"] == "batch" or case["nx"] * case["ny"] * case["nz"] <= 1 << 23


def run(state):
    case, ctxs = state["case"], state["ctxs"]
    if case["kind"] == "batch":
        state["batch"].step(case["steps"])
        xv = [c.read_mesh() for c in ctxs]
        return {"X": np.concatenate([x for x, _ in xv]).astype(np.float32 if case["prec"] != "fp64" else np.float64),
                "V": _keep(case, np.concatenate([v for _, v in xv])),
                "u": [_keep(case, c.read_velocity()) for c in ctxs]}
    c = ctxs[0]
    if case["kind"] == "observe":
        series, n = [], 0
        while n < case["steps"]:
            c.step(10)
            n += 10
            d = c.diagnostics()
            x, v = c.read_mesh()
            for k in range(case["cells"]):
                a = c.object_analyze(k)
                series.append((*a.origin, a.volume, a.area, *a.velocity))
            series.append((d.mass, *d.momentum_fluid, *d.momentum_mesh, 0.0))
        out = {"series": _keep(dict(prec="fp64" if case["prec"] == "fp64" else "fp32"), np.array(series))}
    else:
        c.step(case["steps"])
        x, v = c.read_mesh()
        out = {}
    # positions near 100 moved by 1e-4: FP64 as the library keeps them, FP32 for the forms that compute in it
    out["X"] = x if case["prec"] == "fp64" else torch.from_numpy(x).float()
    out["V"] = _keep(case, v)
    if _reads_velocity(case):
        out["u"] = _keep(case, c.read_velocity())
    return out


def work(case):
    """Bytes and operations of one pass: every stored population read and written once a step, each mesh node's
    position and velocity read and written, and what is handed to the host."""
    b = {"fp64": 8, "fp32": 4, "fp16": 2, "bf16": 2}[case["prec"]]
    r = 8 if case["prec"] == "fp64" else 4
    if case["kind"] == "batch":
        boxes, _ = _boxes(case, 0)
        n, m = sum(x.n_nodes for x in boxes), sum(x.n_mesh_nodes for x in boxes)
    else:
        n, m = case["nx"] * case["ny"] * case["nz"], case["cells"] * NODES[case["mesh"]]
    s = case["steps"]
    reads = s // 10 if case["kind"] == "observe" else 1
    out = reads * 6 * 8 * m + (3 * 8 * n if _reads_velocity(case) else 0)
    return {"bytes": s * (2 * 19 * b * n + m * (48 + 6 * r)) + out, "flops": s * (250.0 * n + 1500.0 * m)}


# ---- the same in 64 bits, in plain torch ---------------------------------------------------------------------------

E = np.array([[0, 0, 0], [1, 0, 0], [-1, 0, 0], [0, 1, 0], [0, -1, 0], [0, 0, 1], [0, 0, -1],
              [1, 1, 0], [-1, -1, 0], [1, -1, 0], [-1, 1, 0], [1, 0, 1], [-1, 0, -1], [1, 0, -1], [-1, 0, 1],
              [0, 1, 1], [0, -1, -1], [0, 1, -1], [0, -1, 1]])
W = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
OPP = [0] + [i + 1 if i % 2 else i - 1 for i in range(1, 19)]


class _Membrane:
    """The cells of one template: relaxed values and the membrane forces of all of them at once."""

    def __init__(self, t, dev):
        self.t = t
        half = {}
        for a, b, c in t.tris.tolist():
            for f, g, w in ((a, b, c), (b, c, a), (c, a, b)):
                half[f, g] = w
        hinge = [(w, f, g, half[g, f]) for (f, g), w in half.items() if f < g]  # (A, B, C, D): the edge is B -> C
        self.h = torch.tensor(hinge, device=dev).T.contiguous()
        self.tri = torch.tensor(t.tris.astype(np.int64), device=dev).T.contiguous()
        x = torch.tensor(t.nodes * np.array(t.stretch), device=dev)[None]
        self.L0 = self.edge(x)[1][0]
        self.th0 = self.angle(x)[0][0]
        n, s = self.area(x)
        self.S0, self.Sg0, self.V0 = s[0], s.sum(), self.volume(x)[0]
        hs = {}
        for k, (a, b, c) in enumerate(t.tris.tolist()):
            for f, g in ((a, b), (b, c), (c, a)):
                hs.setdefault((min(f, g), max(f, g)), []).append(k)
        two = torch.tensor([hs[b, c] for _, b, c, _ in hinge], device=dev)
        self.hbar = (self.S0[two[:, 0]] + self.S0[two[:, 1]]) / self.L0

    def edge(self, x):
        d = x[:, self.h[2]] - x[:, self.h[1]]
        return d, d.norm(dim=-1)

    def area(self, x):
        a, b, c = (x[:, i] for i in self.tri)
        n = torch.linalg.cross(b - a, c - a)
        l = n.norm(dim=-1)
        return n / l[..., None], 0.5 * l

    def volume(self, x):
        a, b, c = (x[:, i] - x[:, :1] for i in self.tri)
        return -(a * torch.linalg.cross(b, c)).sum((-1, -2)) / 6

    def angle(self, x):
        a, b, c, d = (x[:, i] for i in self.h)
        n1, n2 = torch.linalg.cross(b - a, c - a), torch.linalg.cross(c - d, b - d)
        l1, l2 = n1.norm(dim=-1), n2.norm(dim=-1)
        n1, n2 = n1 / l1[..., None], n2 / l2[..., None]
        e = c - b
        e = e / e.norm(dim=-1, keepdim=True)
        return math.pi + torch.atan2((torch.linalg.cross(n1, n2) * e).sum(-1), (n1 * n2).sum(-1)), n1, n2, l1, l2

    def forces(self, x):
        t, F = self.t, torch.zeros_like(x)
        a, b, c, d = self.h
        e, L = self.edge(x)
        st = (L - self.L0) / self.L0
        lam = 1 + st
        kap = 1.0 if t.linear else (lam ** 0.5 + lam ** -2.5) / (lam + lam ** -3)
        f = (t.ks * kap * st / L)[..., None] * e
        F.index_add_(1, b, f).index_add_(1, c, -f)
        th, n1, n2, l1, l2 = self.angle(x)
        f = t.kb * (th - self.th0) / self.th0
        if t.model == "paper":
            fa, fd = f[..., None] * n1, f[..., None] * n2
            fb = fc = -0.5 * (fa + fd)
        else:  # gradient of the bending energy: wing heights l / L and their feet on the edge
            f = f * self.hbar * L
            fa, fd = (f / l1)[..., None] * n1, (f / l2)[..., None] * n2
            pa = (((x[:, a] - x[:, b]) * e).sum(-1) / L ** 2)[..., None]
            pd = (((x[:, d] - x[:, b]) * e).sum(-1) / L ** 2)[..., None]
            fb, fc = -(1 - pa) * fa - (1 - pd) * fd, -pa * fa - pd * fd
        for i, q in ((a, fa), (b, fb), (c, fc), (d, fd)):
            F.index_add_(1, i, q)
        n, S = self.area(x)
        Sg, V = S.sum(1, keepdim=True), self.volume(x)[:, None]
        k = -t.kal * (S - self.S0) / S - t.kag * (Sg - self.Sg0) / Sg
        cv = -t.kv * (V - self.V0) / self.V0
        p = x[:, self.tri]
        w = p - p.mean(1, keepdim=True)
        l = w.norm(dim=-1, keepdim=True)
        if t.model != "paper":
            l = (l * l).mean(1, keepdim=True).sqrt()
        q = k[:, None, :, None] * w / l - (cv * S)[:, None, :, None] * n[:, None] / 3
        for v in range(3):
            F.index_add_(1, self.tri[v], q[:, v])
        return F


class _Reference:
    def __init__(self, box, x, v, d):
        self.box = box
        dev = self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        self.shape = (box.nz, box.ny, box.nx)
        self.d = torch.zeros((19, *self.shape), dtype=torch.float64, device=dev) if d is None else torch.tensor(d, device=dev)
        self.X, self.V = torch.tensor(x, device=dev), torch.tensor(v, device=dev)
        self.Flast = torch.zeros_like(self.X)
        self.dims = torch.tensor([box.nx, box.ny, box.nz], device=dev)
        self.g = torch.tensor(box.g, dtype=torch.float64, device=dev)
        mem = {k: _Membrane(box.templates[k], dev) for k in sorted({o.tid for o in box.objects})}
        self.groups, off = {k: [] for k in mem}, 0
        for o in box.objects:
            nv = len(box.templates[o.tid].nodes)
            self.groups[o.tid].append(torch.arange(off, off + nv, device=dev))
            off += nv
        self.groups = [(mem[k], torch.stack(v)) for k, v in self.groups.items()]
        # solid nodes and their velocity; by node and direction, where the push that would arrive comes from a solid
        self.solid = None
        if box.boundaries:
            z, y, xx = np.meshgrid(*(np.arange(n) + 0.5 for n in self.shape), indexing="ij")
            r = np.stack([xx, y, z], -1)
            solid, uw = np.zeros(self.shape, bool), np.zeros((3, *self.shape))
            for b in box.boundaries:
                if b.kind == "wall":
                    n = np.array(b.normal, float)
                    at = r @ n / np.linalg.norm(n) - b.dist < 0
                else:
                    s = (r - np.array(b.corner)) @ np.linalg.inv(np.array([b.a, b.b, b.c], float))
                    at = ((s >= 0) & (s <= 1)).all(-1)
                solid |= at
                uw[:, at] = np.array(b.velocity)[:, None]
            self.solid, self.uw = torch.tensor(solid, device=dev), torch.tensor(uw, device=dev)

    def roll(self, a, i):
        s = [(int(E[i][c]), -1 - c) for c in range(3) if E[i][c]]
        return torch.roll(a, [q for q, _ in s], [k for _, k in s]) if s else a

    def velocity(self):
        rho = self.box.rho0 + self.d.sum(0)
        u = (torch.einsum("ic,izyx->czyx", torch.tensor(E, dtype=torch.float64, device=self.dev), self.d)
             + 0.5 * self.g[:, None, None, None]) / rho
        return u if self.solid is None else torch.where(self.solid, self.uw, u)

    def collide(self, F):
        box, d = self.box, self.d
        drho = d.sum(0)
        rho = box.rho0 + drho
        j = [sum(int(E[i][c]) * d[i] for i in range(19) if E[i][c]) for c in range(3)]
        u = [(j[c] + 0.5 * F[c]) / rho for c in range(3)]
        out = torch.empty_like(d)
        if box.mrt is None:
            om, gu = 1 / box.tau, 1 - 0.5 / box.tau
            usq = 1.5 * sum(q * q for q in u)
            uF = 3 * sum(p * q for p, q in zip(u, F))
            for i in range(19):
                eu = sum((int(E[i][c]) * u[c] for c in range(3) if E[i][c]), torch.zeros_like(rho))
                eF = sum((int(E[i][c]) * F[c] for c in range(3) if E[i][c]), torch.zeros_like(rho))
                out[i] = (1 - om) * d[i] + om * W[i] * (drho + rho * (3 * eu + 4.5 * eu * eu - usq)) + \
                    gu * W[i] * (3 * eF - uF + 9 * eu * eF)
            return out
        gs, gb, go, ge = box.mrt
        A, B = {}, {}
        for p in range(3):
            for q in range(p, 3):
                A[p, q] = sum(int(E[i][p] * E[i][q]) * d[i] for i in range(19) if E[i][p] * E[i][q]) - (drho / 3 if p == q else 0)
        N = {k: A[k] - rho * u[k[0]] * u[k[1]] for k in A}
        P = {k: u[k[0]] * F[k[1]] + F[k[0]] * u[k[1]] for k in A}
        tn, tp = (sum(M[c, c] for c in range(3)) / 3 for M in (N, P))
        for k in A:
            iso = k[0] == k[1]
            B[k] = rho * u[k[0]] * u[k[1]] + gs * (N[k] - (tn if iso else 0)) + 0.5 * (1 + gs) * (P[k] - (tp if iso else 0)) + \
                (gb * tn + 0.5 * (1 + gb) * tp if iso else 0)
        ta, tb = (sum(M[c, c] for c in range(3)) / 3 for M in (A, B))

        def even(i, M, tr):
            s = sum(((1 if p == q else 2) * int(E[i][p] * E[i][q]) * M[p, q] for p, q in M if E[i][p] * E[i][q]), -tr)
            return W[i] * (drho + 4.5 * s)

        out[0] = even(0, B, tb) + ge * (d[0] - even(0, A, ta))
        for i in range(1, 19, 2):
            e0, e1 = even(i, A, ta), even(i, B, tb)
            o0 = 3 * W[i] * sum(int(E[i][c]) * j[c] for c in range(3) if E[i][c])
            o1 = 3 * W[i] * sum(int(E[i][c]) * (j[c] + F[c]) for c in range(3) if E[i][c])
            ev = e1 + ge * (0.5 * (d[i] + d[i + 1]) - e0)
            od = o1 + go * (0.5 * (d[i] - d[i + 1]) - o0)
            out[i], out[i + 1] = ev + od, ev - od
        return out

    def stream(self, post):
        box, new = self.box, torch.empty_like(post)
        for i in range(19):
            new[i] = self.roll(post[i], i)
            back = post[OPP[i]]
            if self.solid is not None and i:
                val = back - 6 * W[i] * box.rho0 * sum(
                    (-int(E[i][c]) * self.roll(self.uw[c], i) for c in range(3) if E[i][c]), torch.zeros_like(back))
                new[i] = torch.where(self.roll(self.solid, i), val, new[i])
            if box.walls_z and E[i][2]:
                k = 0 if E[i][2] > 0 else box.nz - 1
                new[i][k] = back[k]
        return new if self.solid is None else torch.where(self.solid, self.d, new)

    def repulsion(self, x):
        """Soft-sphere pairs by a sorted cell list (cells of at least the cutoff)."""
        s, L = self.box.repulsion[0], self.dims.double()
        w = x - L * torch.floor(x / L)
        nc = torch.floor(L / max(s.cutoff, 1.0)).long()
        ci = torch.minimum((w / L * nc).long(), nc - 1)
        key = (ci[:, 2] * nc[1] + ci[:, 1]) * nc[0] + ci[:, 0]
        key, order = torch.sort(key)
        F = torch.zeros_like(x)
        for off in np.ndindex(3, 3, 3):
            o = (ci + torch.tensor(off, device=self.dev) - 1) % nc
            k = (o[:, 2] * nc[1] + o[:, 1]) * nc[0] + o[:, 0]
            lo, hi = torch.searchsorted(key, k), torch.searchsorted(key, k, right=True)
            for q in range(int((hi - lo).max())):
                at = torch.nonzero(lo + q < hi)[:, 0]
                other = order[lo[at] + q]
                r = w[at] - w[other]
                r = r - L * torch.round(r / L)
                d = r.norm(dim=-1)
                hit = (d < s.cutoff) & (other != at)
                r, d, at = r[hit], d[hit], at[hit]
                F.index_add_(0, at, (s.a * s.n * d ** -(s.n + 1) / d)[:, None] * r)
        return F

    def step(self):
        box = self.box
        verlet = box.integrator == "verlet"
        if verlet:
            self.V = self.V + 0.5 * self.Flast
            self.X = self.X + self.V
        x = self.X
        F = torch.zeros_like(x)
        for mem, ids in self.groups:
            F[ids] = mem.forces(x[ids])
        if box.repulsion:
            F += self.repulsion(x)
        s = x - 0.5
        i0 = torch.floor(s)
        ph, i0 = s - i0, i0.long()
        u = self.velocity().reshape(3, -1)
        ui, where = torch.zeros_like(x), []
        for k in range(8):
            c = torch.tensor([k & 1, (k >> 1) & 1, k >> 2], device=self.dev)
            w = torch.where(c.bool(), ph, 1 - ph).prod(-1)
            i = i0 + c
            i = torch.stack([i[:, 0] % box.nx, i[:, 1] % box.ny,
                             i[:, 2].clamp(0, box.nz - 1) if box.walls_z else i[:, 2] % box.nz], -1)
            q = (i[:, 2] * box.ny + i[:, 1]) * box.nx + i[:, 0]
            ui += w[:, None] * u[:, q].T
            where.append((q, w))
        drag = box.friction * (self.V - ui)
        G = torch.zeros((box.n_nodes, 3), dtype=torch.float64, device=self.dev)
        for q, w in where:
            G.index_add_(0, q, w[:, None] * drag)
        F = F - drag
        if verlet:
            self.V, self.Flast = self.V + 0.5 * F, F
        else:
            self.V = self.V + F
            self.X = self.X + self.V
        force = self.g[:, None, None, None] + G.T.reshape(3, *self.shape)
        self.d = self.stream(self.collide(force))


def _analysis(ref):
    (mem, ids), = ref.groups
    x = ref.X[ids]
    n, s = mem.area(x)
    return torch.cat([x.mean(1), mem.volume(x)[:, None], s.sum(1)[:, None], ref.V[ids].mean(1)], -1).cpu().numpy()


def exact(case, seed):
    if case["kind"] != "batch" and case["nx"] * case["ny"] * case["nz"] * case["steps"] > 2.3e9:
        return None  # the two largest runs would take too long
    boxes, rng = _boxes(case, seed)
    out = []
    for b in boxes:
        dx, v, d = _start(b, rng)
        x = np.concatenate([o.origin + b.templates[o.tid].nodes @ np.asarray(o.rot).T for o in b.objects]) + dx
        ref, series = _Reference(b, x, v, d), []
        for n in range(case["steps"]):
            ref.step()
            if case["kind"] == "observe" and n % 10 == 9:
                series += [tuple(r) for r in _analysis(ref)]
                j = [float(sum(int(E[i][c]) * ref.d[i].sum() for i in range(19) if E[i][c])) for c in range(3)]
                series.append((b.n_nodes * b.rho0 + float(ref.d.sum()), *j, *ref.V.sum(0).tolist(), 0.0))
        out.append((ref.X.cpu().numpy(), ref.V.cpu().numpy(), ref.velocity().cpu().numpy(), np.array(series)))
    if case["kind"] == "batch":
        return {"X": np.concatenate([o[0] for o in out]), "V": np.concatenate([o[1] for o in out]), "u": [o[2] for o in out]}
    x, v, u, series = out[0]
    got = {"X": x, "V": v}
    if case["kind"] == "observe":
        got["series"] = series
    if _reads_velocity(case):
        got["u"] = u
    return got
