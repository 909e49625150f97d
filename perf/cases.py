"""The work that a program built on this package has it do, as measurable cases.

A case is one call (or the few calls that belong together) of the Python
binding: a single SSP-RK3 step, a run of steps, a captured run replayed, the
guard fill / residual / stage update called one by one, or a graph of steps
of several pools.  `prepare` makes the state and the forest, `run` makes one
pass, `work` says what a pass cannot do without, and `exact` computes the
same outputs in plain torch, in 64 bits, from the method's definition.

States are the isentropic vortex (strength, centre and mean flow drawn from
the seed) or the point blast; steps advance them in place, as a program does.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2502_12620_amd import dgamr as G

GAMMA, CFL = 1.4, 0.1
EDGE = {2: 2.5, 3: 1.25}  # root edge of the vortex forests


def listed():
    return [
        # a small solve stepped one call at a time: the launches and the host
        # path are the time (4x4 roots of 8^2 cells, single level, degree 1)
        dict(name="step_small", call="step", dim=2, degree=1, n_cell=8, rx=4, ry=4, rz=1, refined=0, steps=1),
        # the benchmark's workload: two-level AMR vortex, 100 leaves of 16^2
        # cells, degree 2, 20 steps replayed from a captured run
        dict(name="graph_amr", call="graph", dim=2, degree=2, n_cell=16, rx=8, ry=8, rz=1, refined=1, steps=20),
        # production-size 2-D runs, far above the last-level cache
        dict(name="run_2d_p1", call="run", dim=2, degree=1, n_cell=16, rx=128, ry=128, rz=1, refined=0, steps=2),
        dict(name="run_2d_p2", call="run", dim=2, degree=2, n_cell=16, rx=64, ry=64, rz=1, refined=0, steps=2),
        # production-size 3-D runs at each degree
        dict(name="run_3d_p1", call="run", dim=3, degree=1, n_cell=8, rx=16, ry=16, rz=16, refined=0, steps=2),
        dict(name="run_3d_p2", call="run", dim=3, degree=2, n_cell=8, rx=16, ry=16, rz=16, refined=0, steps=2),
        dict(name="run_3d_p3", call="run", dim=3, degree=3, n_cell=8, rx=8, ry=8, rz=8, refined=0, steps=2),
        # the point blast: three-level AMR, outflow, positivity limiter,
        # between two regrids' indicator
        dict(name="blast_3d", call="run", dim=3, degree=2, n_cell=8, rx=4, ry=4, rz=4, refined=2, steps=4,
             blast=True),
        # FP32 residual arithmetic on an FP64 state
        dict(name="fp32_3d_p2", call="run", dim=3, degree=2, n_cell=8, rx=12, ry=12, rz=12, refined=0, steps=2,
             fp32=True),
        # body-fitted grids: bilinear roots
        dict(name="mapped_2d_p2", call="run", dim=2, degree=2, n_cell=16, rx=48, ry=48, rz=1, refined=0, steps=2,
             mapped=True),
        # a program's own time integrator: guard fill, residual and stage
        # update called one by one, ragged block size and root grid
        dict(name="staged_2d_p3", call="staged", dim=2, degree=3, n_cell=12, rx=52, ry=47, rz=1, refined=1, steps=1),
        # many independent solves batched: one pool per degree, one graph
        dict(name="pools_2d", call="pools", n_cell=16, forests=72, max_roots=128, steps=3),
    ]


# update cost of one cell and stage relative to the others (measured once,
# only used to keep drawn cases below the largest listed one)
_COST = {(2, 1): 1.0, (2, 2): 2.2, (2, 3): 7.0, (3, 1): 3.2, (3, 2): 17.0, (3, 3): 75.0}


def draw(rng):
    """One more case: any of the listed kinds, over the degrees, block sizes,
    root grids and refinements they stand for."""
    call = rng.choice(["step", "run", "run", "run", "graph", "staged", "pools"])
    steps = {"step": 1, "run": rng.randint(1, 3), "graph": rng.randint(3, 20), "staged": 1, "pools": rng.randint(2, 4)}
    n = steps[call]
    if call == "pools":
        return dict(call=call, n_cell=rng.choice([8, 12, 16]), forests=rng.randint(5, 72),
                    max_roots=rng.randint(8, 160), steps=n)
    dim = rng.choice([2, 3])
    p = rng.randint(1, 3)
    fp32 = call == "run" and rng.random() < 0.2
    mapped = call in ("run", "step") and not fp32 and rng.random() < 0.2 and not (dim == 3 and p == 3)
    blast = call == "run" and not mapped and not fp32 and rng.random() < 0.2
    n_cell = rng.choice([4, 6, 8, 10, 12, 16] if dim == 2 else [4, 6, 8])
    # cells per pass, log-uniform, at most three quarters of the largest case's time
    cost = _COST[(dim, p)] * n * (3.0 if mapped else 1.0) * (2.5 if p == 3 and (fp32 or blast) else 1.0)
    top = min(3.0e6, 0.75 * _COST[(3, 2)] * 2 * 2097152 / cost / (2.0 if blast else 1.0))
    cells = math.exp(rng.uniform(math.log(1500.0), math.log(top)))
    k = max(2, int(round((cells / n_cell ** dim) ** (1.0 / dim))))
    rx, ry = max(2, k + rng.randint(-k // 4, k // 4)), max(2, k + rng.randint(-k // 4, k // 4))
    c = dict(call=call, dim=dim, degree=p, n_cell=n_cell, rx=rx, ry=ry, rz=k if dim == 3 else 1,
             refined=0 if rx * ry * k > 4000 else rng.randint(0, 1), steps=n)
    if blast:
        c.update(blast=True, refined=1)
    if fp32:
        c["fp32"] = True
    if mapped:
        c["mapped"] = True
    return c


# ---------------------------------------------------------------- inputs
def _roots(c):
    return (c["rx"], c["ry"], c["rz"])[:c["dim"]]


def _box(c):
    """Lower and upper corner of the domain."""
    if c.get("blast"):
        return [0.0] * c["dim"], [r / max(_roots(c)) for r in _roots(c)]
    return [0.0] * c["dim"], [EDGE[c["dim"]] * r for r in _roots(c)]


def _refine_flags(c, keys, level):
    """+1 for the leaves of `level` whose box touches (blast) or lies near
    the middle of the domain."""
    d, roots = c["dim"], _roots(c)
    lo, hi = _box(c)
    keys = np.asarray(keys)
    tree, lev = keys[:, 0], keys[:, 1]
    near = lev == level
    for a, r in enumerate([tree % roots[0], (tree // roots[0]) % roots[1], tree // (roots[0] * roots[1])][:d]):
        edge = (hi[a] - lo[a]) / roots[a] / 2.0 ** (lev - 1)
        left = lo[a] + r * (hi[a] - lo[a]) / roots[a] + keys[:, 2 + a] * edge
        mid = 0.5 * (lo[a] + hi[a])
        if c.get("blast"):
            near &= (left <= mid + 1e-12) & (mid <= left + edge + 1e-12)
        else:
            near &= abs(left + 0.5 * edge - mid) <= max(0.26 * (hi[a] - lo[a]), 0.51 * edge.max())
    return near.astype(np.int8)


def _nodes(c):
    """Root grid nodes moved by a smooth periodic displacement of 0.1 root."""
    d, roots = c["dim"], _roots(c)
    lo, hi = _box(c)
    axes = [np.linspace(lo[a], hi[a], roots[a] + 1) for a in range(d)]
    grid = np.meshgrid(*axes[::-1], indexing="ij")[::-1]
    nodes = np.stack(grid, axis=-1)
    for a in range(d):
        move = 0.1 * (hi[a] - lo[a]) / roots[a]
        for b in range(d):
            if b != a:
                move = move * np.sin(2.0 * np.pi * (grid[b] - lo[b]) / (hi[b] - lo[b]))
        nodes[..., a] += move
    return nodes


def _pool_members(c):
    """The forests of a pools case: solves of 4 to max_roots roots each, degrees
    1 to 3 (root counts and degrees by the case alone; the states by seed)."""
    rng = np.random.default_rng(c["forests"] * 1009 + c["max_roots"])
    out = []
    for i in range(c["forests"]):
        roots = int(rng.integers(4, c["max_roots"] + 1))
        nx = max(x for x in range(1, math.isqrt(roots) + 1) if roots % x == 0)
        out.append(dict(dim=2, degree=1 + i % 3, n_cell=c["n_cell"], rx=nx, ry=roots // nx, rz=1, refined=0))
    return out


def _flow(c, seed):
    """Parameters of the initial state."""
    rng = np.random.default_rng(seed)
    lo, hi = _box(c)
    if c.get("blast"):
        return dict(p0=1e-5, p1=float(np.exp(rng.uniform(math.log(500.0), math.log(2000.0)))),
                    amp=float(rng.uniform(0.05, 0.2)))
    return dict(eps=float(rng.uniform(1.0, 5.0)), u=float(rng.uniform(0.5, 1.5)), v=float(rng.uniform(0.5, 1.5)),
                w=float(rng.uniform(-0.5, 0.5)), x=float(rng.uniform(lo[0], hi[0])),
                y=float(rng.uniform(lo[1], hi[1])))


def _point_state(c, flow, x, finest):
    """Conserved variables at the points x (a list of d tensors)."""
    d = c["dim"]
    lo, hi = _box(c)
    vel = [torch.zeros_like(x[0]) for _ in range(d)]
    if c.get("blast"):
        inside = torch.ones_like(x[0], dtype=torch.bool)
        for a in range(d):
            inside &= (x[a] - 0.5 * (lo[a] + hi[a])).abs() < finest[a]
        p = torch.where(inside, flow["p1"], flow["p0"])
        rho = 1.0 + flow["amp"] * torch.sin(2.0 * math.pi * x[0]) * torch.cos(2.0 * math.pi * x[1])
    else:
        L = [hi[a] - lo[a] for a in range(2)]
        dx = torch.remainder(x[0] - flow["x"] + 0.5 * L[0], L[0]) - 0.5 * L[0]
        dy = torch.remainder(x[1] - flow["y"] + 0.5 * L[1], L[1]) - 0.5 * L[1]
        r2 = dx * dx + dy * dy
        e1 = torch.exp(0.5 * (1.0 - r2)) * flow["eps"] / (2.0 * math.pi)
        if d == 3:  # a column vortex whose strength varies along it
            e1 = e1 * (1.0 + 0.1 * torch.sin(2.0 * math.pi * (x[2] - lo[2]) / (hi[2] - lo[2])))
            vel[2] = vel[2] + flow["w"]
        vel[0], vel[1] = flow["u"] - e1 * dy, flow["v"] + e1 * dx
        rho = (1.0 - (GAMMA - 1.0) / (2.0 * GAMMA) * e1 * e1) ** (1.0 / (GAMMA - 1.0))
        p = rho ** GAMMA
    ke = sum(v * v for v in vel)
    return [rho] + [rho * v for v in vel] + [p / (GAMMA - 1.0) + 0.5 * rho * ke]


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _initial(c, mesh, seed):
    """The projected initial state, [leaf][var][mode][cell]."""
    b, flow = mesh.basis, _flow(c, seed)
    U = None
    x1, w1 = np.polynomial.legendre.leggauss(c["degree"] + 2)
    for q in np.ndindex(*([len(x1)] * c["dim"])):
        xi = [x1[i] for i in q]
        s = _point_state(c, flow, mesh.points(xi), mesh.finest)
        coef = float(np.prod([w1[i] for i in q])) * b.values([xi])[0] / b.mass
        part = torch.stack(s, 1)[:, :, None, :] * torch.tensor(coef, device=mesh.dev)[None, None, :, None]
        U = part if U is None else U.add_(part)
    return U.contiguous()


# ---------------------------------------------------------------- the passes
def _forest(c):
    d = c["dim"]
    lo, hi = _box(c)
    f = G.Forest(d, c["degree"], c["n_cell"], _roots(c), lo, hi,
                 [G.BC_OUTFLOW if c.get("blast") else G.BC_PERIODIC] * d, 1 + c["refined"], GAMMA,
                 precision=G.FP32 if c.get("fp32") else G.FP64,
                 limiter=G.LIMITER_POSITIVITY if c.get("blast") else G.LIMITER_NONE)
    if c.get("mapped"):
        f.set_root_nodes(_nodes(c))
    for level in range(1, c["refined"] + 1):
        f.adapt(_refine_flags(c, f.keys(), level), f.new_state())
    return f


def prepare(case, seed):
    dt = torch.full((1,), 1e-3, dtype=torch.float64, device="cuda")
    if case["call"] == "pools":
        groups = {}
        for i, m in enumerate(_pool_members(case)):
            groups.setdefault(m["degree"], []).append((m, _forest(m), seed * 1000 + i))
        pools = []
        for p, members in sorted(groups.items()):
            pool = G.Pool(2, p, case["n_cell"], sum(f.n_leaves for _, f, _ in members), len(members))
            for m, f, s in members:
                _, first = pool.admit(f, CFL)
                pool.view(first, f.n_leaves).copy_(_initial(m, _Mesh(m), s))
            pools.append(pool)
        torch.cuda.synchronize()
        return dict(case=case, pools=pools, graph=G.Graph(pools, case["steps"]))
    f = _forest(case)
    u = _initial(case, _Mesh(case, f.keys()), seed)
    s = dict(case=case, f=f, u=u, dt=dt)
    if case["call"] == "staged":
        s.update(un=torch.flip(u, [3]).contiguous(), guard=f.new_guard(), r=f.new_residual(), out=f.new_state())
    else:
        s["work"] = f.new_work()
        if case["call"] == "graph":
            s["graph"] = f.capture_run(u, s["work"], dt, case["steps"], CFL)
    return s


def run(state):
    c = state["case"]
    if c["call"] == "pools":
        state["graph"].launch()
        return [p.u for p in state["pools"]]
    f, u, dt = state["f"], state["u"], state["dt"]
    if c["call"] == "staged":  # the second stage of a step: u_next = 3/4 u_n + 1/4 (u + dt r)
        f.fill_guardcells(u, state["guard"])
        f.dg_residual(u, state["guard"], state["r"])
        f.rk_stage(1, dt, state["un"], u, state["r"], state["out"])
        return dict(guard=state["guard"], r=state["r"], u=state["out"])
    if c["call"] == "graph":
        state["graph"].launch()
    elif c["call"] == "step":
        f.step(u, state["work"], dt, CFL)
    else:
        f.run(u, state["work"], dt, c["steps"], CFL)
    out = dict(u=u, dt=dt)
    if c.get("blast"):
        out["eta"] = f.indicator(u, state["work"])
    return out


def work(case):
    """Bytes: per stage of a state that no cache holds, the stage input read
    and the stage output written once, and the step's base state read in the
    second and third stage (staged: the guard cells, the residual and the
    stage update of one stage).  Operations: evaluation, flux, projection,
    face traces and lifting with the basis' non-zero entries."""
    if case["call"] == "pools":
        total = dict(bytes=0.0, flops=0.0)
        for m in _pool_members(case):
            w = work(dict(m, call="run", steps=case["steps"]))
            total = {k: total[k] + w[k] for k in total}
        return total
    d, p, n = case["dim"], case["degree"], case["n_cell"]
    b, nv = _Basis(d, p), d + 2
    leaves = len(_Mesh(case, device="cpu").level)
    cells = leaves * n ** d
    dof = cells * nv * b.nb
    nnz = lambda m: int(np.count_nonzero(abs(m) > 1e-14))  # noqa: E731
    per_cell = 2 * nv * (nnz(b.vol) + sum(nnz(g) for g in b.dvol)) + len(b.vol) * (20 + 6 * nv * d)
    per_cell += sum(2 * nv * 4 * nnz(b.face[a][1]) + len(b.face[a][1]) * (60 + 10 * nv) for a in range(d))
    if case.get("mapped"):
        per_cell += len(b.vol) * b.nb * (b.nb + 1) + b.nb ** 3 // 3 + 2 * nv * b.nb ** 2
    if case["call"] == "staged":
        guard = leaves * 2 * d * n ** (d - 1) * nv * b.nb * 8.0
        return dict(bytes=dof * 8.0 * 4 + 2 * guard, flops=float(cells) * (per_cell + 4 * nv * b.nb))
    stages = 3.0 * case["steps"]
    return dict(bytes=dof * 8.0 * (2 + 2.0 / 3.0) * stages, flops=float(cells) * (per_cell + 4 * nv * b.nb) * stages)


# ---------------------------------------------------------------- the method in plain torch
class _Basis:
    """Total-degree Legendre products, graded by degree, x exponent
    descending, and their values at the Gauss points of cells and faces."""

    def __init__(self, d, p):
        self.d, self.p = d, p
        modes = [e for e in np.ndindex(*([p + 1] * d)) if sum(e) <= p]
        self.modes = sorted(modes, key=lambda e: (sum(e), [-x for x in e]))
        self.nb = len(self.modes)
        self.mass = np.array([np.prod([2.0 / (2 * e + 1) for e in m]) for m in self.modes])
        x, w = np.polynomial.legendre.leggauss(p + 1)
        idx = [i[::-1] for i in np.ndindex(*([p + 1] * d))]  # x fastest
        self.vpts = [[x[i] for i in q] for q in idx]
        self.vw = np.array([np.prod([w[i] for i in q]) for q in idx])
        self.vol = self.values(self.vpts)
        self.dvol = [self.values(self.vpts, a) for a in range(d)]
        fidx = [i[::-1] for i in np.ndindex(*([p + 1] * (d - 1)))]
        self.fw = np.array([np.prod([w[i] for i in q]) for q in fidx])
        self.fpts = [[self._face(q, x, a, s) for q in fidx] for a in range(d) for s in (-1, 1)]
        self.face = [[self.values(self.fpts[2 * a + k]) for k in (0, 1)] for a in range(d)]
        one = np.zeros((2, p + 1, p + 1))  # halves: P_c((t + s)/2) = sum_a one[.][a][c] P_a(t)
        t, wt = np.polynomial.legendre.leggauss(p + 2)
        for h in (0, 1):
            for a in range(p + 1):
                for c in range(p + 1):
                    one[h, a, c] = 0.5 * (2 * a + 1) * np.sum(
                        wt * self._leg(a, t) * self._leg(c, 0.5 * (t + (1 if h else -1))))
        self.split = np.ones((2 ** d, self.nb, self.nb))
        for ch in range(2 ** d):
            for i, m in enumerate(self.modes):
                for j, n in enumerate(self.modes):
                    self.split[ch, i, j] = np.prod([one[(ch >> a) & 1, m[a], n[a]] for a in range(d)])
        self.comb = np.transpose(self.split, (0, 2, 1)) / self.mass[None, :, None] * self.mass[None, None, :] / 2 ** d

    @staticmethod
    def _leg(n, x):
        return np.polynomial.legendre.Legendre.basis(n)(x)

    @staticmethod
    def _face(q, x, a, s):
        pt = [x[i] for i in q]
        pt.insert(a, float(s))
        return pt

    def values(self, pts, deriv=None):
        out = np.ones((len(pts), self.nb))
        for j, m in enumerate(self.modes):
            for a, e in enumerate(m):
                poly = np.polynomial.legendre.Legendre.basis(e)
                out[:, j] *= (poly.deriv() if a == deriv else poly)(np.array([pt[a] for pt in pts]))
        return out


class _Mesh:
    """Leaves, their geometry and where each guard cell comes from."""

    def __init__(self, c, keys=None, device=None):
        self.c, self.dev = c, device or _device()
        self.d, self.N = c["dim"], c["n_cell"]
        self.basis = _Basis(self.d, c["degree"])
        self.roots = _roots(c)
        self.lo, self.hi = _box(c)
        keys = self._leaves() if keys is None else np.asarray(keys)
        tree, self.level = keys[:, 0], keys[:, 1].astype(np.int64)
        r = np.stack([tree % self.roots[0], (tree // self.roots[0]) % self.roots[1],
                      tree // (self.roots[0] * self.roots[1])], 1)[:, :self.d]
        self.root = r
        self.idx = keys[:, 2:2 + self.d]
        self.block = r * 2 ** (self.level[:, None] - 1) + self.idx  # position at the leaf's level
        size = np.array([(self.hi[a] - self.lo[a]) / self.roots[a] for a in range(self.d)])
        self.finest = list(size / self.N / 2 ** c["refined"])
        self.h = torch.tensor(size[None, :] / self.N / 2.0 ** (self.level[:, None] - 1), device=self.dev)
        n = self.N
        self.ijk = np.stack([a.reshape(-1) for a in np.meshgrid(*([np.arange(n)] * self.d), indexing="ij")][::-1], 0)
        at = self.idx.astype(np.float64) * n  # the leaf's first cell, in cells of its level
        self.cell = [torch.tensor(at[:, a:a + 1], device=self.dev)
                     + torch.tensor(self.ijk[a][None, :].astype(np.float64), device=self.dev) for a in range(self.d)]
        self.width = torch.tensor(1.0 / (n * 2.0 ** (self.level[:, None] - 1)), device=self.dev)  # in roots
        self.nodes = torch.tensor(_nodes(c), device=self.dev) if c.get("mapped") else None

    def _leaves(self):
        """Leaf keys: roots row-major, Morton order inside (x lowest bit)."""
        n = int(np.prod(self.roots))
        keys = np.zeros((n, 5), dtype=np.int64)
        keys[:, 0], keys[:, 1] = np.arange(n), 1
        for level in range(1, self.c["refined"] + 1):
            flags = _refine_flags(self.c, keys, level)
            out = []
            for k, f in zip(keys, flags):
                if not f:
                    out.append(k)
                    continue
                for ch in range(2 ** self.d):
                    kid = np.array([k[0], k[1] + 1, 0, 0, 0])
                    for a in range(self.d):
                        kid[2 + a] = 2 * k[2 + a] + ((ch >> a) & 1)
                    out.append(kid)
            keys = np.array(out)
        return keys

    def _unit(self, xi):
        """Position in the leaf's root, 0 to 1 per axis, of the reference
        point xi of every cell: d tensors [leaf][cell]."""
        return [(self.cell[a] + 0.5 * (xi[a] + 1.0)) * self.width for a in range(self.d)]

    def _corner(self, b):
        """Physical corner b of each leaf's root, [leaf][1][d]."""
        at = [torch.tensor(self.root[:, a] + ((b >> a) & 1), device=self.dev) for a in range(self.d)]
        return self.nodes[tuple(at[::-1])][:, None, :]

    def points(self, xi):
        """Physical coordinates of the reference point xi of every cell."""
        s = self._unit(xi)
        if self.nodes is None:
            edge = [(self.hi[a] - self.lo[a]) / self.roots[a] for a in range(self.d)]
            return [self.lo[a] + edge[a] * (torch.tensor(self.root[:, a:a + 1], device=self.dev) + s[a])
                    for a in range(self.d)]
        x = [0.0] * self.d
        for b in range(2 ** self.d):
            w = math.prod(s[a] if (b >> a) & 1 else 1.0 - s[a] for a in range(self.d))
            for a in range(self.d):
                x[a] = x[a] + w * self._corner(b)[..., a]
        return x

    def metric(self, pts):
        """det J and the rows of adj(J) at the reference points of every
        cell, broadcastable to [leaf][point][cell]."""
        d = self.d
        if self.nodes is None:
            half = [0.5 * self.h[:, a, None, None] for a in range(d)]
            det = math.prod(half)
            return det, [[det / half[e] if a == e else None for a in range(d)] for e in range(d)]
        per = []
        for xi in pts:
            s = self._unit(xi)
            J = [[0.0] * d for _ in range(d)]
            for b in range(2 ** d):
                x = self._corner(b)
                for e in range(d):
                    w = 0.5 * self.width * (1.0 if (b >> e) & 1 else -1.0)
                    for o in range(d):
                        if o != e:
                            w = w * (s[o] if (b >> o) & 1 else 1.0 - s[o])
                    for a in range(d):
                        J[a][e] = J[a][e] + w * x[..., a]
            if d == 2:
                rows = [[J[1][1], -J[0][1]], [-J[1][0], J[0][0]]]
            else:
                rows = [[J[(a + 1) % 3][(e + 1) % 3] * J[(a + 2) % 3][(e + 2) % 3]
                         - J[(a + 1) % 3][(e + 2) % 3] * J[(a + 2) % 3][(e + 1) % 3] for a in range(3)]
                        for e in range(3)]
            det = sum(J[a][0] * rows[0][a] for a in range(d))
            per.append((det, rows))
        det = torch.stack([q[0] for q in per], 1)
        return det, [[torch.stack([q[1][e][a] for q in per], 1) for a in range(d)] for e in range(d)]


class _Solver(_Mesh):
    """Residual, time step, SSP-RK3 step and limiter on the mesh."""

    def __init__(self, c):
        super().__init__(c)
        t = lambda a: torch.tensor(np.ascontiguousarray(a), device=self.dev)  # noqa: E731
        b = self.basis
        self.t = t
        self.B = t(b.vol)
        self.P = [t((b.vw[:, None] * g).T) for g in b.dvol]
        self.F = [[t(b.face[a][k]) for k in (0, 1)] for a in range(self.d)]
        self.L = [[t((b.fw[:, None] * b.face[a][k]).T) for k in (0, 1)] for a in range(self.d)]
        self.mass = t(b.mass)
        self.det, self.rows = self.metric(b.vpts)
        self.frows = [self.metric(b.fpts[2 * a + k])[1][a] for a in range(self.d) for k in (0, 1)]
        self.sources = [self._sources(a, s) for a in range(self.d) for s in (-1, 1)]

    def _sources(self, a, s):
        """Per guard cell (leaf, t) of face (a, s): lists of (kind, entries,
        leaf, cell, operator)."""
        N, d = self.N, self.d
        rest = [b for b in range(d) if b != a]
        tt = [g.reshape(-1) for g in np.meshgrid(*([np.arange(N)] * (d - 1)), indexing="ij")][::-1]
        g = np.zeros((d, len(self.level), N ** (d - 1)), dtype=np.int64)
        for b, ti in zip(rest, tt):
            g[b] = self.block[:, b:b + 1] * N + ti[None, :]
        g[a] = self.block[:, a:a + 1] * N + (N if s > 0 else -1)
        lev = np.broadcast_to(self.level[:, None], g.shape[1:])
        ext = np.array(self.roots)[:, None, None] * 2 ** (lev[None] - 1) * N
        outside = (g[a] < 0) | (g[a] >= ext[a])
        closed = outside if self.c.get("blast") else np.zeros_like(outside)
        g = np.mod(g, ext)
        top = int(self.level.max()) + 1
        ids = {}
        for q in range(0, top + 2):
            shape = [int(r * 2 ** max(q - 1, 0)) for r in self.roots]
            ids[q] = np.full(shape, -1, dtype=np.int64)
            at = np.nonzero(self.level == q)[0]
            ids[q][tuple(self.block[at, b] for b in range(d))] = at

        def look(gc, levels):
            leaf = np.full(levels.shape, -1, dtype=np.int64)
            for q in np.unique(levels):
                m = (levels == q) & (q >= 1)
                leaf[m] = ids[int(q)][tuple(gc[b][m] // N for b in range(d))]
            return leaf

        def cell(gc):
            return sum((gc[b] % N) * N ** b for b in range(d))

        same = look(g, lev)
        coarse = look(g // 2, lev - 1)
        out = []
        own = sum((g[b] % N) * N ** b if b != a else (N - 1 if s > 0 else 0) * N ** a for b in range(d))
        here = np.broadcast_to(np.arange(len(self.level))[:, None], lev.shape)

        def add(mask, leaf, c, op):
            if mask.any():
                at = np.nonzero(mask)
                out.append(tuple(torch.tensor(v, device=self.dev) for v in (at[0], at[1], leaf[mask], c[mask])) + (op,))

        b = self.basis
        sign = np.diag([(-1.0) ** m[a] for m in b.modes])
        add(closed, here, np.broadcast_to(own, lev.shape), self.t(sign))
        add(~closed & (same >= 0), same, cell(g), None)
        is_c = ~closed & (same < 0) & (coarse >= 0)
        child = sum((g[q] % 2) << q for q in range(d))
        for ch in range(2 ** d):
            add(is_c & (child == ch), coarse, cell(g // 2), self.t(b.split[ch]))
        fine = ~closed & (same < 0) & (coarse < 0)
        if fine.any():
            for ch in range(2 ** d):
                gf = np.stack([2 * g[q] + ((ch >> q) & 1) for q in range(d)])
                add(fine, look(gf, lev + 1), cell(gf), self.t(b.comb[ch]))
        return out

    def guard(self, U, a, k):
        """Guard coefficients of face (a, k), [leaf][var][mode][t]."""
        out = torch.zeros(U.shape[0], self.N ** (self.d - 1), U.shape[1], U.shape[2], dtype=U.dtype, device=U.device)
        for i, j, leaf, c, op in self.sources[2 * a + k]:
            v = U[leaf, :, :, c]
            out[i, j] += v if op is None else torch.matmul(v, op.T.contiguous())
        return out.permute(0, 2, 3, 1).contiguous()

    def neighbour(self, U, a, k):
        """Coefficients of the cell across face (a, k) of every cell."""
        N, d = self.N, self.d
        V = U.reshape(*U.shape[:3], *([N] * d))
        W = torch.roll(V, -1 if k else 1, dims=-1 - a)
        W.select(V.dim() - 1 - a, N - 1 if k else 0).copy_(
            self.guard(U, a, k).reshape(*U.shape[:3], *([N] * (d - 1))))
        return W.reshape(U.shape)

    def _dot(self, U, n):
        return sum(U[:, 1 + a] * n[a] for a in range(self.d) if n[a] is not None)

    def pressure(self, U):
        return (GAMMA - 1.0) * (U[:, -1] - 0.5 * sum(U[:, 1 + a] ** 2 for a in range(self.d)) / U[:, 0])

    def flux(self, U, n, p):
        """F(U) . n"""
        un = self._dot(U, n) / U[:, 0]
        F = [U[:, 0] * un]
        for a in range(self.d):
            F.append(U[:, 1 + a] * un if n[a] is None else U[:, 1 + a] * un + p * n[a])
        return torch.stack(F + [(U[:, -1] + p) * un], 1), un

    def residual(self, U):
        R = torch.zeros_like(U)
        S = torch.matmul(self.B, U)
        p = self.pressure(S)
        for e in range(self.d):
            R += torch.matmul(self.P[e], self.flux(S, self.rows[e], p)[0])
        for a in range(self.d):
            for k in (0, 1):
                L = torch.matmul(self.F[a][k], U)
                Q = torch.matmul(self.F[a][1 - k], self.neighbour(U, a, k))
                N = [None if x is None else x * (1.0 if k else -1.0) for x in self.frows[2 * a + k]]
                size = torch.sqrt(sum(x * x for x in N if x is not None))
                n = [None if x is None else x / size for x in N]
                pl, pq = self.pressure(L), self.pressure(Q)
                fl, ul = self.flux(L, n, pl)
                fq, uq = self.flux(Q, n, pq)
                speed = torch.maximum(ul.abs() + torch.sqrt((GAMMA * pl / L[:, 0]).clamp(min=0.0)),
                                      uq.abs() + torch.sqrt((GAMMA * pq / Q[:, 0]).clamp(min=0.0)))
                phi = 0.5 * (fl + fq - speed[:, None] * (Q - L)) * size[:, None]
                R -= torch.matmul(self.L[a][k], phi)
        if self.nodes is None:
            return R / (self.det[:, None] * self.mass[None, None, :, None])
        return self._solve(R)

    def _solve(self, R):
        """M^-1 R with each cell's mass matrix, by elimination."""
        nb, wd = self.basis.nb, self.det * self.t(self.basis.vw)[None, :, None]
        M = [[(wd * (self.B[:, m] * self.B[:, n])[None, :, None]).sum(1) for n in range(nb)] for m in range(nb)]
        R = [R[:, :, m] for m in range(nb)]
        for k in range(nb):
            for r in range(k + 1, nb):
                f = M[r][k] / M[k][k]
                for n in range(k + 1, nb):
                    M[r][n] = M[r][n] - f * M[k][n]
                R[r] = R[r] - f[:, None] * R[k]
        for r in range(nb - 1, -1, -1):
            for n in range(r + 1, nb):
                R[r] = R[r] - M[r][n][:, None] * R[n]
            R[r] = R[r] / M[r][r][:, None]
        return torch.stack(R, 2)

    def time_step(self, U):
        if self.nodes is None:
            m, rows, det = U[:, :, 0], None, None
        else:
            wd = self.det * self.t(self.basis.vw)[None, :, None]
            m = (torch.matmul(self.B, U) * wd[:, None]).sum(2) / wd.sum(1)[:, None]
            det, rows = self.metric([[0.0] * self.d])
        c = torch.sqrt(GAMMA * self.pressure(m) / m[:, 0])
        rate = 0.0
        for e in range(self.d):
            if rows is None:
                rate = rate + ((m[:, 1 + e] / m[:, 0]).abs() + c) / self.h[:, e, None]
            else:
                A = [x[:, 0] for x in rows[e]]
                size = torch.sqrt(sum(x * x for x in A))
                un = sum(m[:, 1 + a] * A[a] for a in range(self.d)) / m[:, 0] / size
                rate = rate + (un.abs() + c) * size / (2.0 * det[:, 0])
        return CFL / rate.max()

    def limit(self, U):
        """Zhang-Shu scaling about the cell mean at the volume, face and
        interior Lobatto points."""
        b = self.basis
        pts = list(b.vpts) + [pt for face in b.fpts for pt in face]
        if b.p == 3:
            pts += [[0.0 if q == a else x for q, x in enumerate(pt)] for a in range(self.d) for pt in b.fpts[2 * a + 1]]
        B = self.t(b.values(pts))
        U = U.clone()
        mean = U[:, :, 0]
        pm = self.pressure(mean)
        eps = torch.minimum(torch.minimum(torch.full_like(pm, 1e-13), mean[:, 0]), pm)
        low = torch.minimum(torch.matmul(B, U[:, 0]).amin(1), mean[:, 0])
        th = torch.where(low < mean[:, 0], ((mean[:, 0] - eps) / (mean[:, 0] - low)).clamp(max=1.0), 1.0)
        U[:, 0, 1:] *= th[:, None]
        p = self.pressure(torch.matmul(B, U))
        t = torch.where(p < eps[:, None], ((pm - eps)[:, None] / (pm[:, None] - p)).clamp(0.0, 1.0), 1.0).amin(1)
        U[:, :, 1:] *= t[:, None, None]
        return U

    def step(self, U, limiter):
        dt = self.time_step(U)
        V = U
        for a, b in ((0.0, 1.0), (0.75, 0.25), (1.0 / 3.0, 2.0 / 3.0)):
            V = a * U + b * (V + dt * self.residual(V))
            if limiter:
                V = self.limit(V)
        return V, dt

    def indicator(self, U):
        """Largest over smallest density mean of a block and its guards."""
        rho = [U[:, 0, 0]] + [self.guard(U, a, k)[:, 0, 0] for a in range(self.d) for k in (0, 1)]
        rho = torch.cat(rho, 1)
        return rho.amax(1) / rho.amin(1)


def exact(case, seed):
    """What `run` returns for these inputs, by the definitions above."""
    if case["call"] == "pools":
        groups = {}
        for i, m in enumerate(_pool_members(case)):
            s = _Solver(m)
            U = _initial(m, s, seed * 1000 + i)
            for _ in range(case["steps"]):
                U, _ = s.step(U, False)
            groups.setdefault(m["degree"], []).append(U)
        return [torch.cat(groups[p]) for p in sorted(groups)]
    s = _Solver(case)
    U = _initial(case, s, seed)
    if case["call"] == "staged":
        un = torch.flip(U, [3])
        guard = torch.stack([s.guard(U, a, k) for a in range(s.d) for k in (0, 1)], 1)
        r = s.residual(U)
        return dict(guard=guard, r=r, u=0.75 * un + 0.25 * (U + 1e-3 * r))
    dt = None
    for _ in range(case["steps"]):
        U, dt = s.step(U, bool(case.get("blast")))
    out = dict(u=U, dt=dt.reshape(1))
    if case.get("blast"):
        out["eta"] = s.indicator(U)
    return out
