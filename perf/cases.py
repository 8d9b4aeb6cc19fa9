"""Timed cases of the droplet runs: what programs of this package have it do.

A program makes a lattice (or a batch of them), advances it some hundreds of
steps, reads the fields it looks at, and goes on.  One pass is one such
round, through the binding's public calls: ``Lattice.step`` and
``Lattice.read``; ``Batch.step``, then ``reduce`` and ``read`` of every member
as the serving loop samples them; ``Lattice.consistent_init`` and a read.

The fields a lattice holds are FP32, so a pass keeps what it read as FP32
tensors.  ``exact`` steps the same inputs in 64 bits with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2212_01617_amd import frelbm as F
from paper_2212_01617_amd import synth
from paper_2212_01617_amd.params import derive_params

# The largest listed case in cell updates; a drawn case stays below it.
MOST_UPDATES = 512 * 256 * 128 * 200
# cell updates that 64-bit torch takes in about ten seconds
MOST_EXACT = 2.0e9


def _solo(name, kind, shape, flow, steps, fields, storage="fp32", ternary=False):
    nx, ny, nz = shape
    return {"name": name, "path": "solo", "kind": kind, "nx": nx, "ny": ny, "nz": nz, "flow": flow, "steps": steps,
            "fields": fields, "storage": storage, "ternary": ternary}


def listed():
    return [
        # The smallest call: the 100 x 100 static drop, watched every few
        # steps (an interactive run, a monitor): launches and the read-back.
        _solo("rest2d_100", 2, (100, 100, 1), "rest", 16, "phi"),
        # The 400 x 200 drop in shear between moving walls, with all that a
        # plot of the flow needs.
        _solo("shear2d_400x200", 2, (400, 200, 1), "shear", 500, "rho,phi,u"),
        # A drop in a ragged box (no multiple of 64), half-precision storage.
        _solo("shear2d_333x150_fp16", 2, (333, 150, 1), "shear", 300, "phi", "fp16"),
        # The small copy of the 3D shear run, the size of tests and trials.
        _solo("shear3d_64x32x32", 3, (64, 32, 32), "shear", 300, "rho,phi,u"),
        # The benchmark's lattice, FP32 and FP16, between two samples.
        _solo("shear3d_256x128x128", 3, (256, 128, 128), "shear", 400, "rho,phi,u"),
        _solo("shear3d_256x128x128_fp16", 3, (256, 128, 128), "shear", 400, "phi", "fp16"),
        # Half the linear size of the breakup campaign's long box (480 x 150
        # x 150), stored in halves rounded stochastically, as it was run.
        _solo("shear3d_240x75x75_fp16_sr", 3, (240, 75, 75), "shear", 300, "phi", "fp16_stochastic"),
        # The four-roller cell: solid bodies, links into moving walls.
        _solo("rollers3d_256x256x64", 3, (256, 256, 64), "rollers", 200, "phi,u"),
        # A third component with its own population.
        _solo("ternary3d_256x128x128", 3, (256, 128, 128), "shear", 150, "phi,psi", ternary=True),
        # A lattice far beyond the caches.
        _solo("shear3d_512x256x128", 3, (512, 256, 128), "shear", 200, "phi"),
        # The serving loop: drops of both kinds, flows and precisions in one
        # batch, one chunk of steps, then every member checked and sampled.
        {"name": "batch_mixed_8", "path": "batch", "members": 8, "size2": 128, "size3": 64, "steps": 200},
        # Consistent initialisation before a run.
        {"name": "init3d_128x64x64", "path": "init", "kind": 3, "nx": 128, "ny": 64, "nz": 64, "flow": "shear",
         "steps": 200, "fields": "rho,phi,u", "storage": "fp32", "ternary": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the same paths, flows, precisions and fields over the
    sizes between the smallest and the largest listed, odd ones among them."""
    what = rng.choice(["2d", "2d", "3d", "3d", "3d", "rollers", "ternary", "batch", "init"])
    if what == "batch":
        return {"path": "batch", "members": rng.randint(2, 16), "size2": rng.randint(64, 200),
                "size3": rng.randint(33, 72), "steps": rng.randint(50, 200)}
    storage = rng.choice(["fp32", "fp32", "fp16", "fp16_stochastic"])
    fields = rng.choice(["phi", "phi,u", "rho,phi,u"])
    kind, flow = 3, "shear"
    if what == "2d":
        kind, flow = 2, rng.choice(["rest", "shear", "rollers"])
        nx, ny, nz = _log_int(rng, 80, 512), _log_int(rng, 60, 256), 1
        if flow == "rest":
            fields = "phi"  # u is at rounding level there
        if flow == "rollers":
            ny = nx
    elif what == "rollers":
        flow = "rollers"
        nx = ny = _log_int(rng, 64, 256)
        nz = _log_int(rng, 24, 96)
    else:
        nx, ny, nz = _log_int(rng, 64, 512), _log_int(rng, 32, 256), _log_int(rng, 32, 128)
    ternary = what == "ternary"
    if ternary:
        storage, fields = "fp32", "phi,psi"
        nx, ny, nz = min(nx, 256), min(ny, 128), min(nz, 128)
    most = min(500, max(16, MOST_UPDATES // (3 * nx * ny * nz)))
    c = _solo("", kind, (nx, ny, nz), flow, 2 * max(1, _log_int(rng, 16, most) // 2) + rng.randint(0, 1), fields,
              storage, ternary)
    del c["name"]
    if what == "init":
        c["path"] = "init"
        c["nx"], c["ny"], c["nz"] = min(nx, 256), min(ny, 128), min(nz, 128)
        c["steps"] = 2 * (1 + min(c["steps"], 200) // 2)
        if c["storage"] == "fp16_stochastic":
            c["storage"] = "fp16"
    return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _inputs(c, seed):
    """Physics, boundaries, mask and initial fields of one lattice: a drop of
    about a fifth of the box (jittered in size and place by the seed) with noise of
    1e-4, in a linear shear between walls normal to the last axis, between
    four rollers along z, or at rest."""
    kind, nx, ny, nz, flow = c["kind"], c["nx"], c["ny"], c["nz"], c["flow"]
    dev = _device()
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    jit = [2.0 * float(v) - 1.0 for v in torch.rand(4, generator=gen, device=dev, dtype=torch.float64).cpu()]
    dims = [nx, ny] if kind == 2 else [nx, ny, nz]
    xi = 2.0
    R = 0.2 * min(dims)
    H, speed = dims[-1], 0.5 * dims[-1]  # wall speed over the shear rate
    if flow == "rollers":
        R = min(0.2 * nx, 0.375 * nz) if kind == 3 else R
        rr = 0.117 * nx
        speed = math.hypot(nx / 4.0, ny / 4.0) - rr  # tip speed over the extension rate
    out = {"shape": (nx, ny, nz), "kind": kind, "bc": (0, 0, 0), "wall_u": np.zeros((3, 2, 3)), "rollers": [],
           "mask": None, "u0": None, "ternary": None}
    if flow == "rest":
        out["phys"] = dict(A=0.04, kappa=0.09, tau_f=1.0, tau_g=1.0, M=0.1)
        xi = 1.5
    else:
        # Re as in the benchmarks, less where a flat box would need walls or rollers faster than 0.05
        dp = derive_params(Re=min(0.5, 0.05 * 6.0 * R * R / speed), Ca=0.1, radius=R, xi=xi, H=float(H),
                           Pe=0.43 if c["path"] != "batch" else 10.0)
        out["phys"] = dp.phys()
    z, y, x = torch.meshgrid(*(torch.arange(n, device=dev, dtype=torch.float64) for n in (nz, ny, nx)), indexing="ij")
    if flow == "shear":
        wall = kind - 1
        out["bc"] = tuple(int(a == wall) for a in range(3))
        out["wall_u"][wall, 0, 0], out["wall_u"][wall, 1, 0] = -dp.wall_u, dp.wall_u
        u0 = torch.zeros((3, nz, ny, nx), device=dev, dtype=torch.float64)
        u0[0] = dp.rate * ((y if kind == 2 else z) - (H - 1) / 2.0)
        out["u0"] = u0.cpu().numpy()
    elif flow == "rollers":
        cs, signs = synth.four_roller_geometry(nx, ny, rr, nz=nz)
        om = dp.rate * speed / rr
        out["rollers"] = [(q, s * om, 2, rr) for q, s in zip(cs, signs)]
        out["mask"] = synth.roller_mask((nz, ny, nx), cs, rr)
    place = [(n - 1) / 2.0 + 0.02 * n * j for n, j in zip((nx, ny, nz), jit)]
    r2 = (x - place[0]) ** 2 + (y - place[1]) ** 2
    if kind == 3:
        r2 = r2 + (z - place[2]) ** 2
    noise = torch.rand(r2.shape, generator=gen, device=dev, dtype=torch.float64)
    phi = torch.tanh((R * (1.0 + 0.05 * jit[3]) - r2.sqrt()) / (math.sqrt(2.0) * xi)) + 2e-4 * (noise - 0.5)
    if c.get("ternary"):
        # a drop of component 1 in a mixture of the other two
        c1 = 0.5 * (1.0 + phi)
        psi = 0.3 * (1.0 - c1)
        phi = c1 - (1.0 - c1 - psi)
        out["psi0"] = psi.cpu().numpy()
        ph = out["phys"]
        out["ternary"] = (4.0 * ph["A"], ph["M"] / 3.0, ph["tau_g"])
    out["phi0"] = phi.cpu().numpy()
    return out


def _member(c, k):
    """Member k of a batch: kinds, flows and precisions in turn, sizes around
    the batch's."""
    kind, flow = (2, 3)[k % 2], ("shear", "rollers")[(k // 2) % 2]
    n = (c["size2"] if kind == 2 else c["size3"]) + (0, 16, -8, 5)[(k // 4) % 4]
    nx, ny, nz = ((2 * n, n, 1) if kind == 2 else (2 * n, n, n)) if flow == "shear" else ((n, n, 1) if kind == 2 else (n, n, n))
    return {"path": "batch", "kind": kind, "nx": nx, "ny": ny, "nz": nz, "flow": flow,
            "storage": ("fp32", "fp16")[(k // 3) % 2], "ternary": False}


def _lattice(c, i, stream):
    p = F.make_params(F.FRE_D2Q9 if c["kind"] == 2 else F.FRE_D3Q19, i["shape"],
                      storage=F.FRE_FP32 if c["storage"] == "fp32" else F.FRE_FP16, bc=i["bc"], wall_u=i["wall_u"],
                      rollers=i["rollers"], ternary=i["ternary"], stochastic_rounding=c["storage"] == "fp16_stochastic",
                      **i["phys"])
    return F.Lattice(p, i["phi0"], None, i["u0"], i["mask"], stream=stream, psi0=i.get("psi0"))


def prepare(case, seed):
    stream = torch.cuda.Stream()
    if case["path"] == "batch":
        members = [_member(case, k) for k in range(case["members"])]
        lats = [_lattice(m, _inputs(m, 1000 * seed + k), stream) for k, m in enumerate(members)]
        needs = [F.Batch.needs(L) for L in lats]
        batch = F.Batch(len(lats), sum(w for w, _ in needs), sum(f for _, f in needs), stream=stream)
        for L in lats:
            batch.add(L)
        return {"case": case, "batch": batch, "lattices": lats}
    i = _inputs(case, seed)
    s = {"case": case, "lattice": _lattice(case, i, stream)}
    if case["path"] == "init":
        s["phi0"], s["u0"] = i["phi0"], i["u0"]
    return s


def _keep(fields):
    return {k: torch.from_numpy(v).float() for k, v in fields.items()}


def run(state):
    c = state["case"]
    if c["path"] == "batch":
        state["batch"].step(c["steps"])
        out = []
        for L in state["lattices"]:
            totals = L.reduce()  # raises if the run went non-finite
            out.append({"totals": torch.from_numpy(totals).float(), **_keep(L.read(("phi",)))})
        return out
    L = state["lattice"]
    if c["path"] == "init":
        L.consistent_init(state["phi0"], state["u0"], c["steps"])
    else:
        L.step(c["steps"])
    return _keep(L.read(tuple(c["fields"].split(","))))


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def _lattice_work(c, steps, values):
    """Every population read once and written once per step at the storage's
    width (FP16 keeps g_0 in FP32), the fields read written once as the host's
    doubles; about 1000 operations for each D3Q19 cell update and half of that
    in D2Q9."""
    q = 9 if c["kind"] == 2 else 19
    cells = c["nx"] * c["ny"] * c["nz"]
    pops = 1 if c["path"] == "init" else (3 if c["ternary"] else 2)
    per = pops * q * 4 if c["storage"] == "fp32" else (q * 2 if pops == 1 else q * 2 + (q - 1) * 2 + 4)
    flops = (1000 if q == 19 else 480) * (pops / 2.0)
    return cells * (steps * 2 * per + 8 * values), cells * steps * flops


def work(case):
    if case["path"] == "batch":
        w = [_lattice_work(_member(case, k), case["steps"], 1) for k in range(case["members"])]
    else:
        w = [_lattice_work(case, case["steps"], sum(3 if f == "u" else 1 for f in case["fields"].split(",")))]
    return {"bytes": float(sum(b for b, _ in w)), "flops": float(sum(f for _, f in w))}


# --------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# --------------------------------------------------------------------------
class _Exact:
    """The free-energy LBM step over whole arrays in float64: two arrays per
    population, streaming by shifts, bounce-back and stencil fills over lists
    of links and of solid cells."""

    def __init__(self, i):
        dev = _device()
        nx, ny, nz = i["shape"]
        axes = 2 if i["kind"] == 2 else 3
        c = [(0, 0, 0)]
        for cz in (-1, 0, 1):
            for cy in (-1, 0, 1):
                for cx in (-1, 0, 1):
                    s = cx * cx + cy * cy + cz * cz
                    if 0 < s <= 2 and not (axes == 2 and cz):
                        c.append((cx, cy, cz))
        wt = {2: (4 / 9, 1 / 9, 1 / 36), 3: (1 / 3, 1 / 18, 1 / 36)}[axes]
        self.c, self.q = c, len(c)
        self.w = [wt[sum(v * v for v in d)] for d in c]
        self.opp = [c.index((-d[0], -d[1], -d[2])) for d in c]
        ph = i["phys"]
        self.k1 = self.k2 = 4.0 * ph["A"]
        self.al2 = ph["kappa"] / (2.0 * ph["A"])
        self.tau = [ph["tau_f"], ph["tau_g"]]
        self.gam = [None, ph["M"] / (ph["tau_g"] - 0.5)]
        self.three = i["ternary"] is not None
        if self.three:
            self.k3, m3, th = i["ternary"]
            self.tau.append(th)
            self.gam.append(m3 / (th - 0.5))
        # one ghost layer at both ends of a wall axis
        pad = i["bc"]
        self.inner = tuple(slice(pad[a], pad[a] + n) for a, n in ((2, nz), (1, ny), (0, nx)))
        ext = tuple(n + 2 * pad[a] for a, n in ((2, nz), (1, ny), (0, nx)))
        code = np.full(ext, 100, np.int64)
        code[self.inner] = 0 if i["mask"] is None else i["mask"]
        self.fluid = torch.from_numpy(code == 0).to(dev)
        self.ff = self.fluid.double()
        n = code.size
        idx = np.arange(n).reshape(ext)
        fluid = code == 0
        nb = [np.roll(idx, (-d[2], -d[1], -d[0]), (0, 1, 2)) for d in c]
        # links of fluid cells into solid ones, with 6 w_i c_i . u_w at the link's middle
        self.links = [None]
        sizes = (ext[2], ext[1], ext[0])
        for k in range(1, self.q):
            at = np.flatnonzero(fluid & ~fluid.reshape(-1)[nb[k]])
            to = nb[k].reshape(-1)[at]
            cw = np.zeros(at.size)
            pos = lambda v: np.stack([v % ext[2], (v // ext[2]) % ext[1], v // (ext[2] * ext[1])], 1)  # noqa: E731
            kinds = code.reshape(-1)[to]
            ghost = kinds == 100
            if ghost.any():
                p = pos(to[ghost])
                acc, cnt = np.zeros((p.shape[0], 3)), np.zeros(p.shape[0])
                for a in range(3):
                    for s in range(2):
                        if pad[a]:
                            on = p[:, a] == (sizes[a] - 1 if s else 0)
                            acc[on] += i["wall_u"][a, s]
                            cnt[on] += 1
                cw[ghost] = (acc / cnt[:, None]) @ np.array(c[k], float)
            for r, (cen, om, _, _) in enumerate(i["rollers"]):
                on = kinds == 2 + r
                if on.any():
                    d = pos(at[on]) - np.array(pad) + 0.5 * np.array(c[k]) - np.array(cen)
                    cw[on] = om * (-d[:, 1] * c[k][0] + d[:, 0] * c[k][1])
            self.links.append((torch.from_numpy(at).to(dev), torch.from_numpy(6.0 * self.w[k] * cw).to(dev))
                              if at.size else None)
        # solid cells next to fluid: the weighted mean over their fluid neighbours
        # (across a wall axis the shifts wrap ghosts onto ghosts only)
        near = np.zeros(n, bool)
        for k in range(1, self.q):
            near |= fluid.reshape(-1)[nb[k].reshape(-1)]
        s = np.flatnonzero(near & ~fluid.reshape(-1))
        self.solid = torch.from_numpy(s).to(dev) if s.size else None
        if s.size:
            tab = np.stack([nb[k].reshape(-1)[s] for k in range(1, self.q)])
            wts = np.array(self.w[1:])[:, None] * fluid.reshape(-1)[tab]
            self.tab = torch.from_numpy(tab).to(dev)
            self.wts = torch.from_numpy(wts / wts.sum(0)).to(dev)

        def grid(v, default):
            out = torch.full(ext, default, dtype=torch.float64, device=dev)
            if v is not None:
                out[self.inner] = torch.from_numpy(np.ascontiguousarray(v)).to(dev)
            return out * self.ff

        self.u0 = [grid(None if i["u0"] is None else i["u0"][a], 0.0) for a in range(3)]
        self.phi0 = grid(i["phi0"], 0.0)
        order = [grid(None, 1.0), self.phi0]
        if self.three:
            order.append(grid(i["psi0"], 0.0))
        mu = self.potentials(order)
        self.p = [torch.stack([self.eq(order[0], self.u0, k) for k in range(self.q)])]
        for a in range(1, len(order)):
            self.p.append(self.order_eq(order[a], mu[a], self.gam[a], self.u0))

    def shift(self, X, k, sign):
        d = self.c[k]
        return torch.roll(X, (sign * d[2], sign * d[1], sign * d[0]), (0, 1, 2))

    def fill(self, X):
        if self.solid is not None:
            X.view(-1)[self.solid] = (X.view(-1)[self.tab] * self.wts).sum(0)
        return X

    def lap(self, X):
        acc = torch.zeros_like(X)
        for k in range(1, self.q):
            acc += self.w[k] * (self.shift(X, k, -1) - X)
        return 6.0 * acc

    def grad(self, X):
        out = [torch.zeros_like(X) for _ in range(3)]
        for k in range(1, self.q):
            s = 3.0 * self.w[k] * self.shift(X, k, -1)
            for a in range(3):
                if self.c[k][a]:
                    out[a] += self.c[k][a] * s
        return out

    def potentials(self, order):
        """mu of rho, phi (and psi) from filled fields, by the concentrations
        C1 = (rho + phi - psi)/2, C2 = (rho - phi - psi)/2, C3 = psi."""
        X = [self.fill(o.clone()) for o in order]
        psi = X[2] if self.three else 0.0
        conc = [0.5 * (X[0] + X[1] - psi), 0.5 * (X[0] - X[1] - psi)] + ([X[2]] if self.three else [])
        kap = [self.k1, self.k2] + ([self.k3] if self.three else [])
        m = [(k * (C * (1 - C) * (1 - 2 * C) - self.al2 * self.lap(C))) * self.ff for k, C in zip(kap, conc)]
        out = [0.5 * (m[0] + m[1]), 0.5 * (m[0] - m[1])]
        if self.three:
            out.append(m[2] - out[0])
        return out

    def dot(self, k, v):
        s = 0.0
        for a in range(3):
            if self.c[k][a]:
                s = s + self.c[k][a] * v[a]
        return s

    def poly(self, u, uu, k):
        cu = self.dot(k, u)
        return 3.0 * cu + 4.5 * cu * cu - 1.5 * uu

    def eq(self, rho, u, k, uu=None):
        uu = sum(v * v for v in u) if uu is None else uu
        return self.w[k] * rho * (1.0 + self.poly(u, uu, k)) * self.ff

    def order_eq(self, X, mu, gam, u):
        uu = sum(v * v for v in u)
        g = torch.stack([self.w[k] * (3.0 * gam * mu + X * self.poly(u, uu, k)) * self.ff for k in range(self.q)])
        g[0] = X - g[1:].sum(0)
        return g

    def moments(self, hold=False):
        order = [p.sum(0) * self.ff for p in self.p]
        if hold:
            order[1] = self.phi0
        mu = self.potentials(order)
        pi = sum(X * m for X, m in zip(order, mu))
        force = [-v for v in self.grad(self.fill(pi))]
        for X, m in zip(order, mu):
            for a, v in enumerate(self.grad(self.fill(X.clone()))):
                force[a] += m * v
        force = [v * self.ff for v in force]
        mom = [sum((self.c[k][a] * self.p[0][k] for k in range(self.q) if self.c[k][a]), torch.zeros_like(pi))
               for a in range(3)]
        inv = torch.where(self.fluid, 1.0 / torch.where(self.fluid, order[0], 1.0), 0.0)
        u = [(m + 0.5 * v) * inv for m, v in zip(mom, force)]
        return order, mu, force, u

    def stream(self, post, X):
        new = torch.empty_like(post)
        new[0] = post[0]
        for k in range(1, self.q):
            new[k] = self.shift(post[k], k, 1)
        for k in range(1, self.q):  # link k of a fluid cell: its own population comes back turned round
            if self.links[k] is not None:
                at, kw = self.links[k]
                new[self.opp[k]].view(-1)[at] = post[k].view(-1)[at] - kw * X.view(-1)[at]
        return new * self.ff

    def step(self, hold=False):
        order, mu, force, u = self.moments(hold)
        if hold:
            u = self.u0
        uu = sum(v * v for v in u)
        uF = sum(a * b for a, b in zip(u, force))
        f, guo = self.p[0], 1.0 - 0.5 / self.tau[0]
        post = torch.empty_like(f)
        for k in range(self.q):
            cu, cF = self.dot(k, u), self.dot(k, force)
            src = guo * self.w[k] * (3.0 * (cF - uF) + 9.0 * cu * cF)
            post[k] = f[k] + (self.eq(order[0], u, k, uu) - f[k]) / self.tau[0] + src
        self.p[0] = self.stream(post, order[0])
        if hold:
            return
        for a in range(1, len(self.p)):
            g = self.p[a]
            self.p[a] = self.stream(g + (self.order_eq(order[a], mu[a], self.gam[a], u) - g) / self.tau[a], order[a])

    def reset_orders(self):
        rho = self.p[0].sum(0) * self.ff
        mu = self.potentials([rho, self.phi0])
        self.p[1] = self.order_eq(self.phi0, mu[1], self.gam[1], self.u0)

    def fields(self, names):
        order, _, _, u = self.moments()
        have = {"rho": order[0], "phi": order[1], "u": None}
        if self.three:
            have["psi"] = order[2]
        cut = lambda X: (X * self.ff)[self.inner].contiguous().cpu()  # noqa: E731
        return {k: torch.stack([cut(v) for v in u]) if k == "u" else cut(have[k]) for k in names}

    def totals(self):
        order, _, _, u = self.moments()
        return torch.tensor([float(order[0].sum()), float(order[1].sum()), float(order[1].abs().sum()),
                             *(float((order[0] * v).sum()) for v in u), 0.0, float(self.ff.sum())], dtype=torch.float64)


def exact(case, seed):
    if case["path"] == "batch":
        members = [_member(case, k) for k in range(case["members"])]
        if sum(m["nx"] * m["ny"] * m["nz"] for m in members) * case["steps"] > MOST_EXACT:
            return None
        out = []
        for k, m in enumerate(members):
            e = _Exact(_inputs(m, 1000 * seed + k))
            for _ in range(case["steps"]):
                e.step()
            out.append({"totals": e.totals(), **e.fields(("phi",))})
        return out
    if case["nx"] * case["ny"] * case["nz"] * case["steps"] > MOST_EXACT:
        return None
    e = _Exact(_inputs(case, seed))
    for _ in range(case["steps"]):
        e.step(hold=case["path"] == "init")
    if case["path"] == "init":
        e.reset_orders()
    return e.fields(tuple(case["fields"].split(",")))
