"""Timed workloads of the library: what a simulation program has it do, through the public entry
points of ``paper_1009_0457_amd.hmc``, from a 16^3 lattice to a 512^3 one.

Kinds of work (a case's ``kind``):

* ``run``       one lattice under load: new spins, a cold stress solve, Monte Carlo sweeps with zone
                solves; returns the spins and the stress field.
* ``zero``      one lattice without load: new spins, sweeps on integer thresholds; returns the spins.
* ``refresh``   one lattice: new spins and a cold stress solve alone (``points`` material points);
                returns the stress field and the macroscopic strain.
* ``ensemble``  independent replicas in one batch, sweeps replayed from captured graphs, a warm
                stress solve before them when loaded; returns every replica's spins (and stress).
* ``gradient``  the stored elastic energy and its derivative with respect to every grain's Euler
                angles and the applied stress, through autograd.
* ``analysis``  grain labels, texture histogram and bond energy of a given microstructure.

Inputs are periodic Voronoi polycrystals with Haar-random orientations, drawn on the device from
the seed.  ``exact`` forms the floating-point results in double precision with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1009_0457_amd import hmc as H

C11, C12, C44 = 246.5, 147.3, 124.7          # nickel, GPa
DEV = "cuda:0"


def _run(name, K, nb, h, nr, Q, load, kT, steps, sweeps=1, proposal=0, screen=0):
    return {"name": name, "kind": "run", "K": K, "neighbors": nb, "h": h, "nr": nr, "Q": Q, "load": load, "kT": kT,
            "steps": steps, "sweeps": sweeps, "proposal": proposal, "screen": screen}


def listed():
    return [
        # the smallest lattice in use: launches and dependent steps, hardly any arithmetic
        _run("run 16 red-black", 16, 6, 1, 50, 8, "z", 0.5, 200),
        # the ordinary loaded run: 5^3 zones x 200 relaxation steps, all 26 neighbours
        _run("run 64", 64, 26, 2, 200, 500, "z", 0.5, 200),
        # the large loaded run the library's headline rate is quoted on, one refresh and one sweep
        _run("run 128", 128, 26, 2, 200, 4000, "xy", 0.7, 200),
        # the widest zone, on an edge that is no multiple of any tile
        _run("run 50 wide zone", 50, 26, 3, 400, 240, "z", 0.7, 100),
        # coarsening without load on a lattice larger than the caches: the colour pass by itself
        {"name": "zero 512", "kind": "zero", "K": 512, "neighbors": 26, "Q": 4000, "kT": 0.7, "sweeps": 4,
         "proposal": 0},
        # grain growth: ten independent 60^3 runs, graph-replayed, latency of many small launches
        {"name": "growth 60 x 10", "kind": "ensemble", "K": 60, "mixed": 0, "n": 10, "neighbors": 26, "h": 2, "nr": 200,
         "Q": 99, "grain_sites": 30, "load": 0.0, "kT": 1.0, "steps": 0, "sweeps": 16, "screen": 0},
        # one sub-load of a texture experiment: ten 100^3 runs, 200 warm steps, one screened sweep
        {"name": "texture 100 x 10", "kind": "ensemble", "K": 100, "mixed": 0, "n": 10, "neighbors": 26, "h": 2,
         "nr": 200, "Q": 91, "grain_sites": 100, "load": 30.0, "kT": 2.6, "steps": 200, "sweeps": 1, "screen": 1},
        # an ensemble of lattices of different sizes under different loads
        {"name": "ensemble 32-96 x 8", "kind": "ensemble", "K": 96, "mixed": 1, "n": 8, "neighbors": 26, "h": 2,
         "nr": 200, "Q": 64, "grain_sites": 512, "load": 200.0, "kT": 0.6, "steps": 200, "sweeps": 1, "screen": 0},
        # the stress solve on a lattice larger than the caches
        {"name": "refresh 512", "kind": "refresh", "K": 512, "points": 1, "Q": 4000, "steps": 20},
        # the stress solve with eight material points per cell
        {"name": "refresh 200 8 points", "kind": "refresh", "K": 200, "points": 8, "Q": 4000, "steps": 100},
        # gradient of the stored energy, at the size and length of the adjoint workload
        {"name": "gradient 64", "kind": "gradient", "K": 64, "Q": 500, "steps": 2000, "every": 50},
        # read-outs between sweeps
        {"name": "analysis 100", "kind": "analysis", "K": 100, "neighbors": 26, "Q": 91, "grain_sites": 100},
    ]


def _even(rng, lo, hi):
    """An even edge, spread over the logarithm of its range."""
    return 2 * int(round(0.5 * math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "zero", "growth", "loaded", "refresh", "refresh8", "gradient", "analysis"])
    if kind == "run":
        h = rng.choice([0, 1, 1, 2, 2, 2, 3])
        K = _even(rng, 2 * h + 10, {0: 128, 1: 128, 2: 100, 3: 48}[h])
        nr = {0: 50, 1: 50, 2: 200, 3: 400}[h] if rng.random() < 0.7 else rng.randrange(20, 300)
        c = _run("", K, rng.choice([6, 26]), h, nr, max(4, K ** 3 // rng.randrange(300, 700)), rng.choice(["z", "xy"]),
                 round(rng.uniform(0.3, 1.0), 3), rng.randrange(10, 200), 1, rng.choice([0, 0, 0, 1]),
                 rng.choice([0, 0, 1]))
        if c["proposal"]:
            c["K"] = min(K, 40)
    elif kind == "zero":
        K = _even(rng, 32, 512)
        c = {"kind": "zero", "K": K, "neighbors": rng.choice([6, 26]), "Q": min(4000, max(8, K ** 3 // 400)),
             "kT": round(rng.uniform(0.3, 1.0), 3), "sweeps": rng.randrange(1, 5), "proposal": rng.choice([0, 0, 1])}
    elif kind == "growth":
        K = _even(rng, 24, 100)
        c = {"kind": "ensemble", "K": K, "mixed": 0, "n": rng.randrange(2, 11), "neighbors": rng.choice([6, 26]), "h": 1,
             "nr": 50, "Q": 99, "grain_sites": rng.choice([30, 100, 400]), "load": 0.0,
             "kT": round(rng.uniform(0.5, 1.5), 3), "steps": 0, "sweeps": rng.randrange(2, 17), "screen": 0}
    elif kind == "loaded":
        h = rng.choice([1, 2, 2])
        c = {"kind": "ensemble", "K": _even(rng, 24, 80), "mixed": rng.choice([0, 1]), "n": rng.randrange(2, 8),
             "neighbors": 26, "h": h, "nr": {1: 50, 2: 200}[h], "Q": rng.randrange(20, 100),
             "grain_sites": rng.randrange(100, 600), "load": round(rng.uniform(20, 300), 1),
             "kT": round(rng.uniform(0.3, 2.6), 3), "steps": rng.randrange(20, 200), "sweeps": 1,
             "screen": rng.choice([0, 1])}
    elif kind in ("refresh", "refresh8"):
        p8 = kind == "refresh8"
        K = _even(rng, 16, 320)
        c = {"kind": "refresh", "K": K, "points": 8 if p8 else 1, "Q": min(4000, max(8, K ** 3 // 500)),
             "steps": rng.randrange(10, 200) if K < 160 else rng.randrange(5, 40)}
    elif kind == "gradient":
        K = _even(rng, 16, 72)
        c = {"kind": "gradient", "K": K, "Q": max(4, K ** 3 // 500), "steps": rng.randrange(50, 800),
             "every": rng.randrange(20, 60)}
    else:
        c = {"kind": "analysis", "K": _even(rng, 24, 200), "neighbors": rng.choice([6, 26]), "Q": 91,
             "grain_sites": rng.choice([30, 100, 400])}
    c.pop("name", None)
    return c


# ---- inputs ------------------------------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFF)
    return g


def _euler(g, Q):
    u = torch.rand((Q, 3), generator=g, device=DEV, dtype=torch.float64)
    two_pi = 2.0 * math.pi
    return torch.stack([two_pi * u[:, 0], torch.acos(2.0 * u[:, 1] - 1.0), two_pi * u[:, 2]], dim=1).cpu().numpy()


def _voronoi(g, K, n):
    """Nearest of n random seed points for every site (periodic), int32, x fastest."""
    if K > 200:                                # the grain structure of a smaller lattice, refined
        f = next(f for f in (4, 3, 2, 1) if K % f == 0 and (f == 1 or K // f >= 64))
        if f > 1:
            s = _voronoi(g, K // f, n).view(K // f, K // f, K // f)
            for d in range(3):
                s = s.repeat_interleave(f, dim=d)
            return s.reshape(-1).contiguous()
    pts = torch.rand((n, 3), generator=g, device=DEV) * K
    x = torch.arange(K, device=DEV, dtype=torch.float32)
    d = x[:, None, None] - pts[None]           # (K, n, 3)
    d = d - K * torch.round(d / K)
    d2 = d * d
    out = torch.empty((K, K, K), dtype=torch.int32, device=DEV)
    rows = max(1, min(K, (1 << 26) // (K * n)))
    for z in range(K):
        for y in range(0, K, rows):
            out[z, y:y + rows] = (d2[None, :, :, 0] + (d2[y:y + rows, None, :, 1] + d2[z, None, None, :, 2])).argmin(dim=2)
    return out.reshape(-1)


def _load(kind, g):
    """Applied stress, MPa: uniaxial along z, or biaxial in x and y, a little off either."""
    base = torch.tensor([0.0, 0, 200, 0, 0, 0] if kind == "z" else [150.0, 150, 0, 0, 0, 0], dtype=torch.float64)
    return (base + 5.0 * torch.randn(6, generator=g, device=DEV, dtype=torch.float64).cpu()).numpy()


def _edges(case):
    if not case["mixed"]:
        return [case["K"]] * case["n"]
    return [max(2 * case["h"] + 2, 2 * int(case["K"] * f / 2)) for f in
            [(1.0, 1 / 3, 2 / 3, 1 / 2)[r % 4] for r in range(case["n"])]]


def _inputs(case, seed):
    g = _gen(seed, 17)
    K, kind = case["K"], case["kind"]
    if kind == "ensemble":
        reps = []
        for r, k in enumerate(_edges(case)):
            spins = _voronoi(g, k, max(2, k ** 3 // case["grain_sites"])) % case["Q"]
            n = torch.randn(3, generator=g, device=DEV, dtype=torch.float64)
            n = n / n.norm()
            s = case["load"] * torch.outer(n, n).cpu()
            reps.append({"K": k, "spins": spins, "euler": _euler(g, case["Q"]),
                         "load": np.array([s[0, 0], s[1, 1], s[2, 2], s[1, 2], s[0, 2], s[0, 1]])})
        return {"reps": reps}
    if kind == "analysis":
        spins = _voronoi(g, K, max(2, K ** 3 // case["grain_sites"])) % case["Q"]
        return {"spins": spins, "euler": _euler(g, case["Q"])}
    spins = _voronoi(g, K, case["Q"])
    euler = _euler(g, case["Q"])
    load = _load(case["load"] if kind == "run" else "z", g)
    if kind == "gradient":
        load = (torch.rand(6, generator=g, device=DEV, dtype=torch.float64).cpu().numpy() - 0.5) * 400.0
    return {"spins": spins, "euler": euler, "load": load}


def prepare(case, seed):
    kind, K = case["kind"], case["K"]
    x = _inputs(case, seed)
    if kind == "ensemble":
        common = H.hmc_default_params(K, case["neighbors"], case["h"])
        common.zone_steps = case["nr"]
        common.zone_screen = case["screen"]
        common.refresh_every = 1 << 30         # the stress solves are asked for by the program itself
        reps = []
        for r, q in enumerate(x["reps"]):
            d = H.hmc_default_replica(common, q["K"], case["Q"])
            d.kT = case["kT"]
            d.seed = int(seed) + r + 1
            if case["load"] == 0.0:
                d.lambda_el = 0.0
            for i in range(6):
                d.sigma_MPa[i] = float(q["load"][i])
            reps.append(d)
        b = H.Batch(common, reps, device=DEV)
        for r, q in enumerate(x["reps"]):
            b.set_replica(r, q["euler"], q["spins"].cpu().numpy())
        b.set_graphs(True)
        H.hmc_set_sweep_index(b.ctx, 1)
        if case["load"] != 0.0:
            b.stress_refresh(case["steps"], True)
        b.synchronize()
        return {"case": case, "batch": b}
    p = H.hmc_default_params(K, case.get("neighbors", 26), case.get("h", 2))
    if kind == "run":
        p.zone_steps, p.proposal, p.zone_screen = case["nr"], case["proposal"], case["screen"]
    if kind in ("zero", "analysis"):
        p.lambda_el = 0.0
        p.proposal = case.get("proposal", 0)
    if kind in ("run", "zero"):
        p.kT = case["kT"]
    if kind == "refresh" and case["points"] == 8:
        H.hmc_set_material_points(p, 8)
    p.seed = int(seed) + 1
    lat = H.Lattice(p, case["Q"], device=DEV)
    lat.set_orientations(x["euler"])
    if "load" in x and kind != "gradient":
        lat.set_load(x["load"])
    s = {"case": case, "lat": lat, "spins": x["spins"]}
    if kind == "gradient":
        lat.set_spins(x["spins"])
        s["euler"] = torch.tensor(x["euler"], dtype=torch.float32, requires_grad=True)
        s["load"] = torch.tensor(x["load"], dtype=torch.float32, requires_grad=True)
    if kind == "analysis":
        lat.set_spins(x["spins"])
    torch.cuda.synchronize()
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "ensemble":
        b = s["batch"]
        if case["load"] != 0.0:
            b.stress_refresh(case["steps"], False)
        b.sweep(case["sweeps"])
        out = {"spins": [b.get_spins(r) for r in range(case["n"])]}
        if case["load"] != 0.0:
            out["stress"] = [b.get_stress(r) for r in range(case["n"])]
        return out
    lat = s["lat"]
    if kind == "run":
        lat.set_spins(s["spins"])
        lat.stress_refresh(case["steps"], True)
        lat.set_sweep_index(1)
        lat.sweep(case["sweeps"])
        return {"spins": lat.get_spins(), "stress": lat.get_stress()}
    if kind == "zero":
        lat.set_spins(s["spins"])
        lat.set_sweep_index(1)
        lat.sweep(case["sweeps"])
        return {"spins": lat.get_spins()}
    if kind == "refresh":
        lat.set_spins(s["spins"])
        lat.stress_refresh(case["steps"], True)
        return {"stress": lat.get_stress(), "strain": torch.from_numpy(lat.macro_strain()).float()}
    if kind == "gradient":
        s["euler"].grad = s["load"].grad = None
        U = H.stored_elastic_energy(s["euler"], s["load"], lat, case["steps"], case["every"])
        U.backward()
        return {"energy": U.detach().float(), "euler_grad": s["euler"].grad, "load_grad": s["load"].grad}
    labels, n = lat.grain_labels()
    hist = lat.texture_histogram((1.0, 0.0, 0.0))
    bonds, _ = lat.energy()
    return {"labels": labels, "n": n, "histogram": hist, "bonds": bonds}


# ---- what a pass cannot do without ----------------------------------------------------------
# One explicit step of a lattice's stress solve: every node's u and w read and written, every grain
# id read; per voxel the strain, the stress and the corner forces.
def _solve_work(K, steps, points):
    nodes = K ** 3 // (8 if points == 8 else 1)
    return (48.0 * nodes + 2.0 * K ** 3) * steps + 26.0 * K ** 3, (126.0 * K ** 3 + 12.0 * nodes) * steps


# One sweep: the spins read and written once.  A real flip reads its neighbours' spins and, under
# load, applies its zone's operator (126 operations a voxel, 12 a node) at least as often as a
# disturbance needs to cross the zone and back; about a quarter of the trials of a polycrystal are
# real flips under neighbour proposals, all under uniform ones, and the screen leaves one in eight.
def _sweep_work(K, sweeps, h, loaded, proposal, screen):
    n = float(K ** 3)
    solves = n * (1.0 if proposal else 0.25) * (0.125 if screen else 1.0) * sweeps if loaded else 0.0
    per = (126.0 * (2 * h + 1) ** 3 + 12.0 * (2 * h + 2) ** 3) * 2 * (2 * h + 2)
    return 4.0 * n * sweeps, 100.0 * n * sweeps + solves * per


def work(case):
    kind = case["kind"]
    if kind == "ensemble":
        b = f = 0.0
        for K in _edges(case):
            loaded = case["load"] != 0.0
            x = _sweep_work(K, case["sweeps"], case["h"], loaded, 0, case["screen"])
            y = _solve_work(K, case["steps"], 1) if loaded else (0.0, 0.0)
            b, f = b + x[0] + y[0] + 4.0 * K ** 3 + (24.0 * K ** 3 if loaded else 0.0), f + x[1] + y[1]
        return {"bytes": b, "flops": f}
    K = case["K"]
    if kind == "run":
        x = _sweep_work(K, case["sweeps"], case["h"], True, case["proposal"], case["screen"])
        y = _solve_work(K, case["steps"], 1)
        return {"bytes": x[0] + y[0] + 32.0 * K ** 3, "flops": x[1] + y[1]}
    if kind == "zero":
        x = _sweep_work(K, case["sweeps"], 0, False, 0, 0)
        return {"bytes": x[0] + 8.0 * K ** 3, "flops": x[1]}
    if kind == "refresh":
        x = _solve_work(K, case["steps"], case["points"])
        return {"bytes": x[0] + 28.0 * K ** 3, "flops": x[1]}
    if kind == "gradient":
        x = _solve_work(K, case["steps"], 1)
        return {"bytes": 2.5 * x[0], "flops": 3.5 * x[1]}
    return {"bytes": 2.0 * 3 * K ** 3 + 4.0 * K ** 3, "flops": 60.0 * K ** 3}


# ---- the same results in double precision, with plain torch -----------------------------------
_VOIGT = [(0, 0), (1, 1), (2, 2), (1, 2), (0, 2), (0, 1)]


def _rotation(e):
    c1, s1, c, s, c2, s2 = (f(e[:, k]) for k in range(3) for f in (torch.cos, torch.sin))
    return torch.stack([c1 * c2 - s1 * c * s2, -c1 * s2 - s1 * c * c2, s1 * s,
                        s1 * c2 + c1 * c * s2, -s1 * s2 + c1 * c * c2, -c1 * s,
                        s * s2, s * c2, c], dim=1).view(-1, 3, 3)


def _stiffness(e):
    """(Q, 6, 6) lab-frame stiffness of cubic crystals: C12 d_ij d_kl + C44 (d_ik d_jl + d_il d_jk)
    + (C11 - C12 - 2 C44) sum_m a_im a_jm a_km a_lm."""
    A = _rotation(e)
    P = torch.stack([A[:, i] * A[:, j] for i, j in _VOIGT], dim=1)           # (Q, 6, m)
    iso = torch.zeros((6, 6), dtype=e.dtype, device=e.device)
    iso[:3, :3] += C12
    iso += torch.diag(torch.tensor([2 * C44] * 3 + [C44] * 3, dtype=e.dtype, device=e.device))
    return iso + (C11 - C12 - 2 * C44) * (P[:, :, None, :] * P[:, None, :, :]).sum(-1)


def _sh(t, d):
    """Value one site up along x (0), y (1) or z (2); t is (..., z, y, x)."""
    return torch.roll(t, -1, dims=t.ndim - 1 - d)


def _dn(t, d):
    return torch.roll(t, 1, dims=t.ndim - 1 - d)


class _Solve:
    """Heavy-ball relaxation of the periodic lattice, one material point per voxel."""

    def __init__(self, K, spins, C, Sigma, points=1):
        self.K, self.n3, self.points = K, K ** 3, points
        q = spins.long()
        S = torch.linalg.inv(C)
        cnt = torch.bincount(q, minlength=C.shape[0]).double()
        self.Sigma, self.Smean = Sigma, (cnt[:, None, None] * S).sum(0) / self.n3
        self.q, self.C = q, C
        self.rows = {(i, j): C[:, i, j][q].view(K, K, K) for i in range(6) for j in range(i, 6)}
        lam = max(C11 + 2 * C12, C11 - C12, 2 * C44)
        n = K / 2 if points == 8 else K
        a, b = math.sqrt((8 if points == 8 else 4) * lam), math.sqrt(0.5 * (C11 - C12)) * 2 * math.sin(math.pi / n)
        self.alpha, self.beta = 4 / (a + b) ** 2, ((a - b) / (a + b)) ** 2
        k = K // 2 if points == 8 else K
        self.u = torch.zeros((3, k, k, k), dtype=torch.float64, device=C.device)
        self.E = self.Smean @ Sigma

    def stress(self, e):
        return [sum(self.rows[min(i, j), max(i, j)] * e[j] for j in range(6)) for i in range(6)]

    def _dif(self, t, d):
        """Derivative along d at the voxel centres of a node field."""
        for k in range(3):
            t = (_sh(t, k) - t) if k == d else 0.5 * (_sh(t, k) + t)
        return t

    def _difT(self, t, d):
        for k in range(3):
            t = (_dn(t, k) - t) if k == d else 0.5 * (_dn(t, k) + t)
        return t

    # eight points per cell: sites 2X + p of cell X, weights 3/4 and 1/4 along each axis
    def _up(self, t, d, deriv):
        a, b = t, _sh(t, d)
        lo, hi = (0.5 * (b - a),) * 2 if deriv else (0.75 * a + 0.25 * b, 0.25 * a + 0.75 * b)
        ax = t.ndim - 1 - d
        return torch.stack([lo, hi], dim=ax + 1).flatten(ax, ax + 1)

    def _upT(self, t, d, deriv):
        ax = t.ndim - 1 - d
        lo, hi = t.unflatten(ax, (-1, 2)).unbind(ax + 1)
        if deriv:
            g = 0.5 * (lo + hi)
            return _dn(g, d) - g
        return (0.75 * lo + 0.25 * hi) + _dn(0.25 * lo + 0.75 * hi, d)

    def grad(self, t, d):
        if self.points != 8:
            return self._dif(t, d)
        for k in range(3):
            t = self._up(t, k, k == d)
        return t

    def gradT(self, t, d):
        if self.points != 8:
            return self._difT(t, d)
        for k in range(3):
            t = self._upT(t, k, k == d)
        return t

    def strain(self, u, E):
        g = self.grad
        e = [g(u[0], 0), g(u[1], 1), g(u[2], 2), g(u[1], 2) + g(u[2], 1), g(u[0], 2) + g(u[2], 0), g(u[0], 1) + g(u[1], 0)]
        return [x + E[i] for i, x in enumerate(e)]

    def forces(self, s):
        """sum_v B_v^T s_v."""
        T, row = self.gradT, [(0, 5, 4), (5, 1, 3), (4, 3, 2)]
        return torch.stack([T(s[r[0]], 0) + T(s[r[1]], 1) + T(s[r[2]], 2) for r in row])

    def steps(self, n, keep=None):
        w, wE = torch.zeros_like(self.u), torch.zeros_like(self.E)
        for _ in range(n):
            if keep is not None:
                keep.append((self.u, self.E))
            s = self.stress(self.strain(self.u, self.E))
            mean = torch.stack([x.mean() for x in s])
            w = self.beta * w - self.alpha * self.forces(s)
            wE = self.beta * wE + self.alpha * (self.Sigma - mean)
            self.u, self.E = self.u + w, self.E + wE

    def field(self):
        return torch.stack([x.reshape(-1) for x in self.stress(self.strain(self.u, self.E))])


def _exact_gradient(case, x):
    e = torch.tensor(x["euler"], dtype=torch.float32).double().to(DEV).requires_grad_(True)
    Sig = (torch.tensor(x["load"], dtype=torch.float32).double() * 1e-3).to(DEV)
    C = _stiffness(e)
    m = _Solve(case["K"], x["spins"], C.detach(), Sig)
    kept = []
    m.steps(case["steps"], kept)
    # M accumulates dU/dC per voxel (upper triangle of eta eps^T), S_ the stored-energy terms
    M = {k: torch.zeros_like(v) for k, v in m.rows.items()}

    def add(eta, eps, f):
        for (i, j), a in M.items():
            a.add_(f * (eta[i] * eps[j] + (eta[j] * eps[i] if i != j else 0.0)))

    eps = m.strain(m.u, m.E)
    s = m.stress(eps)
    U = 0.5 * sum((a * b).sum() for a, b in zip(s, eps))
    add(eps, eps, 0.5)
    ub, wb = m.forces(s), torch.zeros_like(m.u)
    Eb = torch.stack([t.sum() for t in s])
    wEb, Sb = torch.zeros_like(Eb), torch.zeros_like(Eb)
    for u, E in reversed(kept):
        wt, wEt = wb + ub, wEb + Eb
        b = m.alpha * wEt
        eta = m.strain(m.alpha * wt, b / m.n3)
        add(eta, m.strain(u, E), -1.0)
        tau = m.stress(eta)
        ub, wb = ub - m.forces(tau), m.beta * wt
        Eb, wEb = Eb - torch.stack([t.sum() for t in tau]), m.beta * wEt
        Sb = Sb + b
    # start: E_0 = mean(S) Sigma
    cnt = torch.bincount(m.q, minlength=case["Q"]).double()
    loss = (((cnt[:, None, None] * torch.linalg.inv(C)).sum(0) / m.n3 @ Sig) * Eb).sum()
    for (i, j), a in M.items():
        per = torch.zeros(case["Q"], dtype=torch.float64, device=DEV).index_add_(0, m.q, a.reshape(-1))
        loss = loss + (per * C[:, i, j]).sum()
    loss.backward()
    return {"energy": U.cpu(), "euler_grad": e.grad.cpu(), "load_grad": (1e-3 * (Sb + m.Smean @ Eb)).cpu()}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("zero", "analysis") or (kind == "ensemble" and case["load"] == 0.0):
        return None
    x = _inputs(case, seed)
    table = lambda e: _stiffness(torch.tensor(e, dtype=torch.float64, device=DEV))  # noqa: E731
    if kind == "ensemble":
        out = []
        for q in x["reps"]:
            m = _Solve(q["K"], q["spins"], table(q["euler"]), torch.tensor(q["load"], device=DEV) * 1e-3)
            m.steps(case["steps"])             # the cold solve of prepare()
            m.steps(case["steps"])             # the warm one of the pass
            out.append(m.field())
        return {"spins": [None] * case["n"], "stress": out}
    if kind == "gradient":
        return _exact_gradient(case, x)
    m = _Solve(case["K"], x["spins"], table(x["euler"]), torch.tensor(x["load"], device=DEV) * 1e-3,
               case.get("points", 1))
    m.steps(case["steps"])
    if kind == "run":
        return {"spins": None, "stress": m.field()}
    return {"stress": m.field(), "strain": m.E.cpu()}
