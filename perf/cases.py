"""What this library's users run, as cases that can be timed: operator applies
on device tensors and whole time steps from state to state.

The sizes are those of the scenarios and of bench.py: the 16^3 cube, design
instances of 32^3 to 96^3 cells, the 128 x 128 x 64 layered aquifer, the pile
field on 256 x 256 x 128 Q1 or 128 x 128 x 64 Q2 cells (8.5 M nodes per field),
the island with its pile columns, and terrain-following hexahedra.

A case is a dict of plain values:

  kind "apply"  one Mesh.apply_operator call: mesh "box", "graded" or "hex",
                degree 1 or 2, field 0 pressure / 1 heat, bits 64 or 32;
  kind "steps"  `steps` backward-Euler steps and both fields' new states, as a
                run that writes its output every few steps: site "cube",
                "aquifer", "island" or "design", mode "fp64", "refined" or
                "learned", `count` meshes advanced as one batch.

`tune` calls autotune while the mesh is set up, as bench.py does.  `exact` is
the same discretisation in plain torch FP64: Gauss quadrature cell by cell, and
Jacobi-preconditioned CG / BiCGStab for the steps.
"""
import math

import numpy as np
import torch

import paper_2103_00081_amd as hts

DAY = 86400.0
T15C = 288.15
RHO_W, MU_W, C_W, LAM_W, G, B_PORO = 1000.0, 1.0e-3, 4.18e6, 0.6, 9.81, 1.0e5
NX, NY, NZ = "nx", "ny", "nz"

EXTENT = {"piles": (1000.0, 1000.0, 200.0), "cube": (100.0, 100.0, 100.0), "aquifer": (500.0, 500.0, 100.0),
          "island": (640.0, 400.0, 100.0), "design": (200.0, 200.0, 200.0), "terrain": (500.0, 500.0, 100.0)}
MODE = {"fp64": hts.MODE_FP64, "refined": hts.MODE_FP32_REFINED, "learned": hts.MODE_LEARNED}


def _apply(name, mesh, degree, n, field, bits, tune):
    return {"name": name, "kind": "apply", "mesh": mesh, "degree": degree, NX: n[0], NY: n[1], NZ: n[2],
            "field": field, "bits": bits, "tune": tune}


def _steps(name, site, degree, n, mode, steps, count, tune, graph):
    return {"name": name, "kind": "steps", "site": site, "degree": degree, NX: n[0], NY: n[1], NZ: n[2],
            "mode": mode, "steps": steps, "count": count, "tune": tune, "graph": graph}


def listed():
    return [
        # the smallest call: one apply on a design instance of the least size
        _apply("apply q1 pressure f32 32^3", "box", 1, (32, 32, 32), 0, 32, False),
        # the layered aquifer's heat operator, the one its FP64 residuals use
        _apply("apply q1 heat f64 128x128x64", "box", 1, (128, 128, 64), 1, 64, True),
        # the pile field at full size: the pressure operator in FP64 and the
        # heat operator in FP32, the two that bench.py reports first
        _apply("apply q1 pressure f64 256x256x128", "box", 1, (256, 256, 128), 0, 64, True),
        _apply("apply q1 heat f32 256x256x128", "box", 1, (256, 256, 128), 1, 32, True),
        # the pile field on Q2 cells, as many nodes
        _apply("apply q2 pressure f32 128x128x64", "box", 2, (128, 128, 64), 0, 32, True),
        # a graded Q2 site mesh with odd cell counts
        _apply("apply q2 heat f64 graded 101x77x33", "graded", 2, (101, 77, 33), 1, 64, False),
        # general hexahedra following the terrain
        _apply("apply hex heat f32 128x128x64", "hex", 1, (128, 128, 64), 1, 32, True),
        # a small study: steady Darcy flow and a heated block, FP64 defaults
        _steps("steps cube fp64 16^3", "cube", 1, (16, 16, 16), "fp64", 10, 1, False, False),
        # the headline workload, ten days between outputs
        _steps("steps aquifer refined 128x128x64", "aquifer", 1, (128, 128, 64), "refined", 10, 1, True, True),
        # the same flow with the network as pressure preconditioner
        _steps("steps aquifer learned 64x64x32", "aquifer", 1, (64, 64, 32), "learned", 4, 1, False, True),
        # a pile site on Q2 cells with odd counts, a working week
        _steps("steps island refined q2 51x33x13", "island", 2, (51, 33, 13), "refined", 5, 1, False, True),
        # design scenarios of different sizes advanced as one batch
        _steps("steps design batch of 8", "design", 1, (48, 48, 48), "refined", 4, 8, False, True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.7:
        mesh = rng.choice(["box", "box", "box", "graded", "hex"])
        degree = 1 if mesh == "hex" else rng.choice([1, 2])
        top = {("hex", 1): 128, ("box", 1): 256, ("graded", 1): 256}.get((mesh, degree), 128)
        nx = _log(rng, 16, top)
        ny = min(top, max(8, int(nx * rng.uniform(0.6, 1.2))))
        nz = min(top // 2, max(8, int(nx * rng.uniform(0.3, 1.0))))
        return _apply("", mesh, degree, (nx, ny, nz), rng.choice([0, 1]), rng.choice([64, 32]), rng.random() < 0.5)
    site = rng.choice(["cube", "aquifer", "island", "design"])
    degree = rng.choice([1, 1, 2]) if site == "island" else 1
    nx = _log(rng, 16, 48 if degree == 2 else 112)
    shape = {"cube": (1.0, 1.0), "design": (1.0, 1.0), "aquifer": (1.0, 0.5), "island": (0.625, 0.25)}[site]
    if site in ("cube", "design"):
        nx = min(nx, 64)
    n = (nx, max(8, int(nx * shape[0])), max(8, int(nx * shape[1])))
    return _steps("", site, degree, n, rng.choice(["fp64", "refined", "refined"]), rng.choice([1, 2, 4, 5]),
                  rng.choice([2, 4, 6]) if site == "design" else 1, rng.random() < 0.3, rng.random() < 0.7)


# ------------------------------------------------------------- problem data
def _tf(c0=0.0, cx=0.0, cy=0.0, cz=0.0, amp=0.0, period=1.0, phase=0.0, kind=0):
    return (kind, c0, cx, cy, cz, amp, period, phase)


def _edges(lo, length, n, swing):
    """n + 1 edges of a smoothly graded axis (cell sizes vary by (1 + swing) : (1 - swing))."""
    s = np.arange(n + 1) / n
    e = lo + length * (s + swing * np.sin(2.0 * np.pi * s) / (2.0 * np.pi))
    e[0], e[-1] = lo, lo + length
    return e


def _terrain(extent, n):
    """Node coordinates of a terrain-following mesh: node planes between a
    curved bottom and top, the interior sheared horizontally."""
    (lx, ly, lz), (nx, ny, nz) = extent, n
    s, v, u = np.meshgrid(np.arange(nz + 1) / nz, np.arange(ny + 1) / ny, np.arange(nx + 1) / nx, indexing="ij")
    pi = np.pi
    top = lz + 8.0 * np.sin(2 * pi * u) * np.sin(pi * v)
    bot = 5.0 * np.cos(pi * u) * np.cos(2 * pi * v)
    x = lx * u + 0.03 * lx * (s - 0.5) * np.sin(pi * u) * np.sin(pi * v)
    y = ly * v + 0.03 * ly * np.sin(2 * pi * u) * np.sin(pi * v) * (1.0 - s)
    return np.stack([x.reshape(-1), y.reshape(-1), (bot + s * (top - bot)).reshape(-1)], axis=1)


def _axis(length, n, degree, edges):
    e = np.arange(n + 1) * (length / n) if edges is None else edges
    if degree == 1:
        return e
    out = np.empty(2 * n + 1)
    out[0::2], out[1::2] = e, 0.5 * (e[:-1] + e[1:])
    return out


def _scenario(site, degree, n, mesh, seed):
    """Geometry, materials, boundary data and initial states; arrays drawn
    from the seed (layered lognormal permeability, scattered porosity)."""
    gen = torch.Generator().manual_seed(int(seed))
    rnd = lambda *shape: torch.rand(*shape, generator=gen, dtype=torch.float64)
    ext = EXTENT[site]
    nx, ny, nz = n
    nc = nx * ny * nz
    sc = {"site": site, "degree": degree, "n": n, "extent": ext, "edges": None, "coords": None, "B": B_PORO,
          "c_w": C_W, "source": None, "lines": [], "cols": [], "bcs": []}
    if mesh == "graded":
        sc["edges"] = [_edges(0.0, ext[d], n[d], (0.5, 0.4, 0.3)[d]) for d in range(3)]
    if mesh == "hex":
        sc["coords"] = _terrain(ext, n)
    layer = np.minimum(np.arange(nz) * 5 // nz, 4)
    means = (-12.0 + 2.0 * rnd(5)).numpy()
    noise = torch.randn(nc, generator=gen, dtype=torch.float32).numpy().reshape(nz, -1)
    sc["perm"] = np.power(10.0, means[layer][:, None] + 0.5 * noise.astype(np.float64)).reshape(-1)
    sc["phi"] = (0.2 + 0.15 * torch.rand(nc, generator=gen, dtype=torch.float32)).double().numpy()
    rg = RHO_W * G
    top = ext[2]
    hyd = _tf(c0=1.0e5 + rg * top, cz=-rg)
    slope = {"piles": 0.001, "island": 5.0 / rg, "design": 0.001, "terrain": 0.005}.get(site, 0.0)
    p0 = _tf(c0=hyd[1] + rg * slope * ext[0], cx=-rg * slope, cz=-rg)
    sc["P0"], sc["T0"] = p0, _tf(T15C)
    sides = (0, 1, 2, 3) if site == "aquifer" else (0, 1)
    sc["bcs"] = [(0, f, 0, p0) for f in sides]
    sc["bcs"] += [(1, f, 0, _tf(T15C)) for f in range(6) if site != "terrain" or f != 4]
    if site == "cube":
        sc["B"] = 0.0
        sc["perm"], sc["phi"] = np.full(nc, 1.0e-12), np.full(nc, 0.3)
        sc["bcs"][0] = (0, 0, 0, _tf(c0=hyd[1] + 1.0e4, cz=-rg))
        src = np.zeros((nz, ny, nx))
        o = [int(float(rnd(1)) * (v - 2)) for v in (nz, ny, nx)]
        src[o[0]:o[0] + 2, o[1]:o[1] + 2, o[2]:o[2] + 2] = 10.0 + 40.0 * float(rnd(1))
        sc["source"] = src.reshape(-1)
    elif site == "aquifer":
        sc["lines"] = [(150.0, 250.0, 0.0, 100.0, 1, _tf(0.01), 313.15), (350.0, 250.0, 0.0, 100.0, 1, _tf(-0.01), 0.0)]
    elif site == "piles":
        ph = (2.0 * math.pi * rnd(400)).tolist()
        sc["lines"] = [(262.5 + 25.0 * (i % 20), 262.5 + 25.0 * (i // 20), 170.0, 200.0, 0,
                        _tf(amp=50.0, period=365.0 * DAY, phase=ph[i], kind=1), 0.0) for i in range(400)]
    elif site == "design":
        pick = torch.randperm(361, generator=gen)[:10 + int(float(rnd(1)) * 190)].sort().values.tolist()
        hot = 303.15 + 20.0 * float(rnd(1))
        sc["cols"] = [(10.0 * (q % 19 + 1), 10.0 * (q // 19 + 1), 170.0, 200.0, _tf(hot)) for q in pick]
    elif site == "island":
        geo = _tf(c0=287.45 + 0.03 * top, cz=-0.03)
        sc["T0"] = geo
        sc["bcs"] = [(0, f, 0, p0) for f in sides] + [(1, f, 0, geo) for f in range(4)]
        sc["bcs"] += [(1, 4, 1, _tf(-0.0891)),
                      (1, 5, 0, _tf(c0=287.45, amp=3.5, period=365.0 * DAY, phase=math.asin(0.2 / 3.5), kind=1))]
        i0, j0 = 4 + int(8 * float(rnd(1))), 4 + int(4 * float(rnd(1)))
        sc["cols"] = [(20.0 * (i0 + i), 20.0 * (j0 + j), 40.0, 100.0, _tf(c0=288.55, amp=13.0, period=365.0 * DAY, kind=2))
                      for j in range(6) for i in range(10)]
    sc["axes"] = [_axis(ext[d], n[d], degree, None if sc["edges"] is None else sc["edges"][d]) for d in range(3)]
    return sc


def _nodes(sc):
    if sc["coords"] is not None:
        return sc["coords"][:, 0], sc["coords"][:, 1], sc["coords"][:, 2]
    z, y, x = np.meshgrid(sc["axes"][2], sc["axes"][1], sc["axes"][0], indexing="ij")
    return x.reshape(-1), y.reshape(-1), z.reshape(-1)


def _wave(tf, t):
    s = math.sin(2.0 * math.pi * t / tf[6] + tf[7])
    return 0.0 if tf[0] == 0 else (s if tf[0] == 1 else (1.0 if s >= 0.0 else -1.0))


def _value(tf, x, y, z, t):
    return tf[1] + tf[2] * x + tf[3] * y + tf[4] * z + tf[5] * _wave(tf, t)


def _mesh(sc, tune):
    m = hts.Mesh((0.0, 0.0, 0.0), sc["extent"], sc["n"], sc["degree"], edges=sc["edges"], coords=sc["coords"])
    nc = m.ncell
    m.set_materials(sc["perm"], sc["phi"], np.full(nc, 2.5), np.full(nc, 2.0e6), RHO_W, MU_W, sc["c_w"], LAM_W, G, sc["B"])
    for field, face, kind, tf in sc["bcs"]:
        m.set_face_bc(field, face, kind, tf)
    if sc["source"] is not None:
        m.set_volume_source(sc["source"])
    for x, y, z0, z1, kind, rate, t_inj in sc["lines"]:
        m.add_line_source(x, y, z0, z1, kind, rate, t_inj)
    for x, y, z0, z1, tf in sc["cols"]:
        m.add_dirichlet_column(1, x, y, z0, z1, tf)
    return m


# --------------------------------------------------------- prepare and run
def _apply_site(case):
    return "terrain" if case["mesh"] == "hex" else "piles"


def _apply_data(case, seed):
    """Scenario, pressure state and operand of one operator apply."""
    sc = _scenario(_apply_site(case), case["degree"], (case[NX], case[NY], case[NZ]), case["mesh"], seed)
    x, y, z = _nodes(sc)
    gen = torch.Generator().manual_seed(int(seed) + 7)
    # drawdown and mounding of up to 2 m of water about the regional gradient
    p = _value(sc["P0"], x, y, z, 0.0) + 2.0e4 * (torch.rand(x.size, generator=gen, dtype=torch.float32).numpy() - 0.5)
    u = torch.randn(x.size, generator=gen, dtype=torch.float32)
    return sc, p, u if case["bits"] == 32 else u.double()


def _batch_sizes(case):
    """Cells per instance: a batch holds instances of 2/3 to 4/3 of the size."""
    c = case["count"]
    if c == 1:
        return [(case[NX], case[NY], case[NZ])]
    f = [2.0 / 3.0 + (2.0 / 3.0) * i / (c - 1) for i in range(c)]
    return [tuple(max(8, int(round(case[k] * v))) for k in (NX, NY, NZ)) for v in f]


def prepare(case, seed):
    if case["kind"] == "apply":
        sc, p, u = _apply_data(case, seed)
        m = _mesh(sc, case["tune"])
        m.set_state(hts.PRESSURE, p, 0.0)
        if case["tune"]:
            hts.autotune([m])
        u = u.cuda()
        return {"case": case, "mesh": m, "x": u, "y": torch.zeros_like(u)}
    meshes = []
    for i, n in enumerate(_batch_sizes(case)):
        sc = _scenario(case["site"], case["degree"], n, "box", seed + 1000 * i)
        m = _mesh(sc, case["tune"])
        x, y, z = _nodes(sc)
        m.set_state(hts.PRESSURE, _value(sc["P0"], x, y, z, 0.0) * np.ones(m.nnode), 0.0)
        m.set_state(hts.TEMPERATURE, _value(sc["T0"], x, y, z, 0.0) * np.ones(m.nnode), 0.0)
        meshes.append(m)
    if case["tune"]:
        hts.autotune(meshes)
    o = hts.default_opts(mode=MODE[case["mode"]], use_graph=int(case["graph"]), rtol=1e-8,
                         mg_coarse_max=600 if case["count"] > 1 else 5000)
    state = {"case": case, "meshes": meshes, "opts": o}
    if case["mode"] == "learned":
        net = hts.Net(levels=4, channels=(16, 32, 48, 64), seed=int(seed) % 65521)
        o.nn = net.h.value
        state["net"] = net
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "apply":
        state["mesh"].apply_operator(case["field"], hts.FP64 if case["bits"] == 64 else hts.FP32, DAY, state["x"], state["y"])
        return state["y"]
    hts.advance(state["meshes"], case["steps"], DAY, state["opts"])
    return [{"P": m.get_state(hts.PRESSURE)[0], "T": m.get_state(hts.TEMPERATURE)[0]} for m in state["meshes"]]


def work(case):
    """Bytes: node vectors and per-cell coefficients in and out once.  Flops:
    the sum-factorised element products (per cell: Q1 140 pressure and 390
    heat, Q2 1460 and 3500, general hexahedra 1300 and 2600); of a step, one
    application of either field's operator, which no solver can do without."""
    per = {1: (140.0, 390.0), 2: (1460.0, 3500.0), 3: (1300.0, 2600.0)}
    if case["kind"] == "apply":
        d, b, heat = case["degree"], case["bits"] // 8, case["field"] == 1
        cells = case[NX] * case[NY] * case[NZ]
        nodes = (d * case[NX] + 1) * (d * case[NY] + 1) * (d * case[NZ] + 1)
        hexa = case["mesh"] == "hex"
        vectors, coefs = (3, 3) if heat else (2, 1)
        return {"bytes": b * (vectors * nodes + coefs * cells) + (24 * nodes if hexa else 0),
                "flops": per[3 if hexa else d][case["field"]] * cells}
    total = {"bytes": 0.0, "flops": 0.0}
    for n in _batch_sizes(case):
        d = case["degree"]
        cells = n[0] * n[1] * n[2]
        nodes = (d * n[0] + 1) * (d * n[1] + 1) * (d * n[2] + 1)
        total["bytes"] += case["steps"] * 8.0 * (4 * nodes + 3 * cells)
        total["flops"] += case["steps"] * (per[d][0] + per[d][1]) * cells
    return total


# -------------------------------------------------------------------- exact
def _basis(p, x):
    """Values and derivatives of the 1D Lagrange basis at x (numpy array)."""
    if p == 1:
        return np.stack([1 - x, x], 1), np.stack([-np.ones_like(x), np.ones_like(x)], 1)
    return (np.stack([(2 * x - 1) * (x - 1), 4 * x * (1 - x), x * (2 * x - 1)], 1),
            np.stack([4 * x - 3, 4 - 8 * x, 4 * x - 1], 1))


class _Fem:
    """The discretisation by (p + 1)^3-point Gauss quadrature, cell by cell, in
    FP64: node vectors [NZ, NY, NX], cell data [ncell]."""

    def __init__(self, sc, device):
        self.p, self.n, self.dev = sc["degree"], sc["n"], device
        p = self.p
        g, w = np.polynomial.legendre.leggauss(p + 1)
        g, w = 0.5 * (g + 1.0), 0.5 * w
        b, d = _basis(p, g)
        kron = lambda z, y, x: np.einsum("za,yb,xc->zyxabc", z, y, x).reshape((p + 1) ** 3, -1)
        dv = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=device)
        # [quantity][point][local node]: value and the three reference derivatives
        self.B = dv(np.stack([kron(b, b, b), kron(b, b, d), kron(b, d, b), kron(d, b, b)]))
        self.w = dv(np.einsum("z,y,x->zyx", w, w, w).reshape(-1))
        self.nq, self.nl = (p + 1) ** 3, (p + 1) ** 3
        self.shape = tuple(p * v + 1 for v in reversed(self.n))
        self.ncell = self.n[0] * self.n[1] * self.n[2]
        if sc["coords"] is None:
            h = [dv(np.diff(sc["axes"][k][::p])) for k in range(3)]
            hz, hy, hx = torch.meshgrid(h[2], h[1], h[0], indexing="ij")
            self.ih = [1.0 / v.reshape(-1) for v in (hx, hy, hz)]
            self.detw = self.w[:, None] * (hx * hy * hz).reshape(-1)[None]
            self.inv = None
        else:
            xyz = dv(sc["coords"].T.copy()).reshape(3, *self.shape)
            # J[i][j] = d x_i / d xi_j at the points
            J = [[self.B[1 + j] @ self.gather(xyz[i]) for j in range(3)] for i in range(3)]
            cof = lambda i, j: (J[(i + 1) % 3][(j + 1) % 3] * J[(i + 2) % 3][(j + 2) % 3]
                                - J[(i + 1) % 3][(j + 2) % 3] * J[(i + 2) % 3][(j + 1) % 3])
            det = sum(J[0][j] * cof(0, j) for j in range(3))
            self.detw = self.w[:, None] * det
            self.inv = [[cof(i, j) / det for j in range(3)] for i in range(3)]   # d xi_j / d x_i

    def _views(self, u):
        p, (nx, ny, nz) = self.p, self.n
        for a in range(p + 1):
            for b in range(p + 1):
                for c in range(p + 1):
                    yield u[a:a + p * nz - p + 1:p, b:b + p * ny - p + 1:p, c:c + p * nx - p + 1:p]

    def gather(self, u):
        return torch.stack([v.reshape(-1) for v in self._views(u)])

    def scatter(self, w):
        y = torch.zeros(self.shape, dtype=torch.float64, device=self.dev)
        for a, v in enumerate(self._views(y)):
            v += w[a].reshape(v.shape)
        return y

    def grad(self, U, i):
        """d/dx_i at the points."""
        if self.inv is None:
            return (self.B[1 + i] @ U) * self.ih[i]
        return sum((self.B[1 + j] @ U) * self.inv[i][j] for j in range(3))

    def grad_t(self, s, i):
        """sum_q s_q dN_a/dx_i."""
        if self.inv is None:
            return self.B[1 + i].T @ (s * self.ih[i])
        return sum(self.B[1 + j].T @ (s * self.inv[i][j]) for j in range(3))

    def flux(self, P, k):
        """Darcy flux -k (grad P + rho_w g e_z) at the points."""
        U = self.gather(P)
        return [-k * (self.grad(U, i) + (RHO_W * G if i == 2 else 0.0)) for i in range(3)]

    def apply(self, u, mass, stiff, adv=0.0, q=None):
        U = self.gather(u)
        g = [self.grad(U, i) for i in range(3)]
        v = 0.0
        if mass is not None:
            v = mass * (self.B[0] @ U)
        if q is not None:
            v = v + adv * sum(q[i] * g[i] for i in range(3))
        W = sum(self.grad_t(stiff * self.detw * g[i], i) for i in range(3))
        if mass is not None or q is not None:
            W = W + self.B[0].T @ (self.detw * v)
        return self.scatter(W)

    def diagonal(self, mass, stiff):
        W = sum((self.B[1 + i] ** 2).T @ (stiff * self.detw * self.ih[i] ** 2) for i in range(3))
        if mass is not None:
            W = W + (self.B[0] ** 2).T @ (mass * self.detw)
        return self.scatter(W)


def _constrained(sc, field, t, dev):
    """Mask and values of the constrained nodes, [NZ, NY, NX]."""
    x, y, z = (np.asarray(v).reshape([sc["degree"] * v2 + 1 for v2 in reversed(sc["n"])]) for v in _nodes(sc))
    mask, g = np.zeros(x.shape, bool), np.zeros(x.shape)
    for f, face, kind, tf in sc["bcs"]:
        if f == field and kind == 0:
            at = [slice(None)] * 3
            at[2 - face // 2] = 0 if face % 2 == 0 else -1
            at = tuple(at)
            mask[at], g[at] = True, _value(tf, x[at], y[at], z[at], t)
    if field == 1:
        for cx, cy, z0, z1, tf in sc["cols"]:
            # the nearest node column, the higher one on a tie
            i, j = (int(a.size - 1 - np.argmin(np.abs(a - v)[::-1].round(9))) for a, v in ((sc["axes"][0], cx), (sc["axes"][1], cy)))
            za = sc["axes"][2]
            ks = np.nonzero((za >= z0 - 1e-9 * sc["extent"][2]) & (za <= z1 + 1e-9 * sc["extent"][2]))[0]
            mask[ks, j, i], g[ks, j, i] = True, _value(tf, cx, cy, 0.0, t)
    return torch.tensor(mask, device=dev), torch.tensor(g, device=dev)


def _coefficients(sc, dev):
    dv = lambda a: torch.tensor(a, dtype=torch.float64, device=dev)
    phi = sc["phi"]
    return dv(sc["perm"] / MU_W), dv((1 - phi) * 2.5 + phi * LAM_W), dv((1 - phi) * 2.0e6 + phi * sc["c_w"])


def _exact_apply(case, seed, dev):
    sc, p, u = _apply_data(case, seed)
    fem = _Fem(sc, dev)
    k, lam, cT = _coefficients(sc, dev)
    x = u.to(dev, torch.float64).reshape(fem.shape)
    mask, _ = _constrained(sc, case["field"], DAY, dev)
    xm = torch.where(mask, torch.zeros_like(x), x)
    if case["field"] == 0:
        y = fem.apply(xm, torch.ones_like(k), DAY * sc["B"] * k)
    else:
        q = fem.flux(torch.tensor(p, device=dev).reshape(fem.shape), k)
        y = fem.apply(xm, cT, DAY * lam, DAY * sc["c_w"], q)
    return torch.where(mask, x, y).reshape(-1)


def _line_points(sc, line, dev):
    """Quadrature along a line source: node indices and shape values
    [points, nl], weights [points]."""
    p, (nx, ny, nz) = sc["degree"], sc["n"]
    x, y, z0, z1 = line[:4]
    loc = []
    for d, v in ((0, x), (1, y)):
        e = sc["axes"][d][::p]
        c = min(max(int(np.searchsorted(e, v, side="right")) - 1, 0), sc["n"][d] - 1)
        loc.append((c, _basis(p, np.array([(v - e[c]) / (e[c + 1] - e[c])]))[0][0]))
    gp, gw = np.polynomial.legendre.leggauss(p + 1)
    e, ids, sh, wt = sc["axes"][2][::p], [], [], []
    for c in range(nz):
        a, b = max(z0, e[c]), min(z1, e[c + 1])
        if b <= a:
            continue
        for q in range(p + 1):
            zq = a + (b - a) * 0.5 * (gp[q] + 1.0)
            bz = _basis(p, np.array([(zq - e[c]) / (e[c + 1] - e[c])]))[0][0]
            sh.append(np.einsum("a,b,c->abc", bz, loc[1][1], loc[0][1]).reshape(-1))
            zi, yi, xi = (p * c + np.arange(p + 1), p * loc[1][0] + np.arange(p + 1), p * loc[0][0] + np.arange(p + 1))
            ids.append((xi[None, None] + (p * nx + 1) * (yi[None, :, None] + (p * ny + 1) * zi[:, None, None])).reshape(-1))
            wt.append(0.5 * gw[q] * (b - a))
    return (torch.tensor(np.array(ids), device=dev), torch.tensor(np.array(sh), device=dev), torch.tensor(wt, dtype=torch.float64, device=dev))


def _krylov(A, dinv, b, x, symmetric, tol=1e-13, most=6000):
    """Jacobi-preconditioned CG, or BiCGStab, to a relative residual tol."""
    dot = lambda u, v: float((u * v).sum())
    stop = tol * math.sqrt(dot(b, b))
    r = b - A(x)
    if symmetric:
        z = dinv * r
        d, rz = z.clone(), dot(r, z)
        for _ in range(most):
            if math.sqrt(dot(r, r)) <= stop:
                break
            q = A(d)
            a = rz / dot(d, q)
            x, r = x + a * d, r - a * q
            z = dinv * r
            rz, old = dot(r, z), rz
            d = z + (rz / old) * d
        return x
    r0, rho, a, w = r.clone(), 1.0, 1.0, 1.0
    v = d = torch.zeros_like(r)
    for _ in range(most):
        if math.sqrt(dot(r, r)) <= stop:
            break
        rho, old = dot(r0, r), rho
        d = r + (rho / old) * (a / w) * (d - w * v)
        dh = dinv * d
        v = A(dh)
        a = rho / dot(r0, v)
        s = r - a * v
        sh = dinv * s
        t = A(sh)
        w = dot(t, s) / max(dot(t, t), 1e-300)
        x, r = x + a * dh + w * sh, s - w * t
    return x


def _exact_steps(sc, steps, dev):
    fem = _Fem(sc, dev)
    k, lam, cT = _coefficients(sc, dev)
    x, y, z = _nodes(sc)
    at = lambda tf: torch.tensor(_value(tf, x, y, z, 0.0) * np.ones(x.size), device=dev).reshape(fem.shape)
    P, T = at(sc["P0"]), at(sc["T0"])
    lines = [(ln, _line_points(sc, ln, dev)) for ln in sc["lines"]]
    one, steady = torch.ones_like(k), sc["B"] <= 0.0
    s = 1.0 if steady else DAY * sc["B"]
    mass = None if steady else one
    gravity = fem.scatter(fem.grad_t(-s * RHO_W * G * k * fem.detw, 2))
    source = None
    if sc["source"] is not None:
        source = fem.scatter(fem.B[0].T @ (fem.detw * torch.tensor(sc["source"], device=dev)))
    # nodal weights of a unit flux through the bottom
    cell = {1: (0.5, 0.5), 2: (1 / 6, 2 / 3, 1 / 6)}[sc["degree"]]
    wall = []
    for d in range(2):
        a, p = sc["axes"][d], sc["degree"]
        v = np.zeros(a.size)
        for i, h in enumerate(np.diff(a[::p])):
            v[p * i:p * i + p + 1] += h * np.array(cell)
        wall.append(torch.tensor(v, device=dev))
    area = wall[1][:, None] * wall[0][None]

    def solve(A, diag, b, field, t, x0, symmetric):
        mask, g = _constrained(sc, field, t, dev)
        zero = torch.zeros_like(g)
        b = torch.where(mask, zero, b - A(g))
        reduced = lambda u: torch.where(mask, u, A(torch.where(mask, zero, u)))
        dinv = torch.where(mask, torch.ones_like(g), 1.0 / diag)
        return g + _krylov(reduced, dinv, b, torch.where(mask, zero, x0), symmetric)

    for n in range(steps):
        t = (n + 1) * DAY
        b = gravity if steady else gravity + fem.apply(P, one, torch.zeros_like(k))
        b = b.clone()
        for ln, (ids, sh, wt) in lines:
            if ln[4] == 1:
                b.view(-1).index_add_(0, ids.reshape(-1), (s * _value(ln[5], 0, 0, 0, t) / (ln[3] - ln[2]) * wt[:, None] * sh).reshape(-1))
        P = solve(lambda u: fem.apply(u, mass, s * k), fem.diagonal(mass, s * k), b, 0, t, P, True)
        q = fem.flux(P, k)
        b = fem.apply(T, cT, torch.zeros_like(k))
        if source is not None:
            b = b + DAY * source
        for field, face, kind, tf in sc["bcs"]:
            if field == 1 and kind == 1:
                b[0] += -DAY * tf[1] * area
        wells = []
        for ln, (ids, sh, wt) in lines:
            rate = _value(ln[5], 0, 0, 0, t)
            if ln[4] == 0:
                b.view(-1).index_add_(0, ids.reshape(-1), (DAY * rate * wt[:, None] * sh).reshape(-1))
            elif rate > 0.0:
                c = DAY * C_W * rate / (ln[3] - ln[2]) * wt
                wells.append((ids, sh, c))
                b.view(-1).index_add_(0, ids.reshape(-1), (c[:, None] * sh * ln[6]).reshape(-1))

        def heat(u):
            out = fem.apply(u, cT, DAY * lam, DAY * sc["c_w"], q)
            for ids, sh, c in wells:
                at_points = (u.reshape(-1)[ids] * sh).sum(1)
                out.view(-1).index_add_(0, ids.reshape(-1), (c[:, None] * at_points[:, None] * sh).reshape(-1))
            return out

        T = solve(heat, fem.diagonal(cT, DAY * lam), b, 1, t, T, False)
    return P.reshape(-1), T.reshape(-1)


def exact(case, seed):
    dev = "cuda"
    if case["kind"] == "apply":
        return _exact_apply(case, seed, dev)
    out = []
    for i, n in enumerate(_batch_sizes(case)):
        sc = _scenario(case["site"], case["degree"], n, "box", seed + 1000 * i)
        P, T = _exact_steps(sc, case["steps"], dev)
        out.append({"P": P, "T": T})
    return out
