"""Performance cases: the work that programs built on this library have it do.

A case is one system (or a batch of systems) that a user keeps on the GPU and
advances: a pass runs a few time steps through `Lattice.step` / `Batch.step`
and reads the new state back, densities, velocity and owner map into the
user's device tensors, particle states to the host, as the studies in this
package do between blocks of steps (`adsorption.trajectory`,
`coarsening.history`) and as the benchmark does around its timed region.

Fields and particle velocities and forces are recorded in the form's own
storage type (a run that keeps its populations in half precision keeps its
snapshots in half precision); positions and orientations stay in double.

`exact` is the same time step written down plainly in torch, in double, with
none of this package's code.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1109_3277_amd.binding import Batch, Lattice
from paper_1109_3277_amd.workloads import place_particles, shoemake_quaternions, tilt_quaternion

DTYPE = {"fp64": torch.float64, "fp32": torch.float32, "fp16_dev": torch.float16, "bf16_dev": torch.bfloat16}
STORE = {"fp64": 8, "fp32": 4, "fp16_dev": 2, "bf16_dev": 2}


def _case(name, nx, ny, nz, precision, steps, **more):
    c = dict(name=name, nx=nx, ny=ny, nz=nz, precision=precision, steps=steps, tau=1.0, g_br=0.08, psi=1,
             fields="mixture", particles="none", phi=0.0, tile=0, walls="none", pairs=False, density=8.0, domain_size=False,
             systems=0)
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: one step of the single ellipsoid at an interface, its
        # state read after every step (a trajectory sampled at full rate)
        _case("interface_step", 32, 32, 64, "fp64", 1, fields="layers", particles="one"),
        # the adsorption study of Sec. 4: walls, one ellipsoid, sampled every 50 steps
        _case("adsorption_64", 64, 64, 64, "fp64", 50, g_br=0.1, fields="lamellae", particles="one", walls="resting"),
        # a sheared channel of ragged size with Psi = rho
        _case("channel_ragged_f32", 90, 53, 74, "fp32", 20, g_br=0.02, psi=0, walls="moving"),
        # phase separation without particles: the two sizes and forms of the
        # domain-growth study, L(t) read as it goes
        _case("spinodal_128_f64", 128, 128, 128, "fp64", 20, domain_size=True),
        _case("spinodal_256_f32", 256, 256, 256, "fp32", 20, domain_size=True),
        # a mixture of other viscosity (tau not 1) with coloured ellipsoids on a ragged box
        _case("ragged_tau125_f64", 150, 87, 101, "fp64", 5, tau=1.25, particles="mixed", phi=0.08, pairs=True, density=20.0),
        # a lower viscosity without particles, single precision
        _case("spinodal_192_tau08_f32", 192, 192, 192, "fp32", 10, tau=0.8),
        # the bijel of Sec. 4 at its size, as the study runs it: pair terms on, L(t) read
        _case("bijel_256_f64", 256, 256, 256, "fp64", 10, particles="prolate", phi=0.15, tile=4, pairs=True,
              domain_size=True),
        # the bijel in the reduced form of half storage
        _case("bijel_256_f16", 256, 256, 256, "fp16_dev", 10, particles="prolate", phi=0.15, tile=4),
        # polydisperse coloured ellipsoids: the benchmark's domain in its other two
        # reduced forms, and in double at the largest size
        _case("mixed_384_f32", 384, 384, 384, "fp32", 10, particles="mixed", phi=0.1, tile=3),
        _case("mixed_512_f64", 512, 512, 320, "fp64", 10, particles="mixed", phi=0.1, tile=4),
        # the ensemble: many small uneven systems advanced as one batch
        _case("ensemble_f32", 0, 0, 0, "fp32", 20, fields="layers", particles="one", systems=48),
    ]


def draw(rng):
    """One more case of the listed ranges: any form, boxes from a few thousand
    nodes to some 20 million, odd and ragged sides, with and without
    particles, walls and pair terms, or a batch."""
    prec = rng.choice(["fp64", "fp32", "fp16_dev", "bf16_dev"])
    tau = 1.0 if rng.random() < 0.7 else rng.choice([1.25, 1.5])
    if rng.random() < 0.2:
        return _unnamed(_case("", 0, 0, 0, prec, rng.randint(2, 20), tau=tau, fields="layers", particles="one",
                              density=20.0, systems=rng.randint(2, 48)))
    rep = rng.choice([1, 1, 2, 2, 3])
    side = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    kind = rng.choice(["none", "one", "prolate", "mixed"])
    lo = 24 if kind in ("none", "one") else 40
    dims = [side(lo, 96) * rep for _ in range(3)]
    c = _case("", *dims, prec, rng.randint(1, 12), tau=tau, particles=kind, tile=rep if kind in ("prolate", "mixed") else 0)
    if kind in ("prolate", "mixed"):
        # bodies that are not kept apart collide in long runs: pair terms on
        c.update(phi=round(rng.uniform(0.04, 0.12), 3), pairs=True, density=20.0)
    if kind == "one":
        c.update(fields="layers", walls=rng.choice(["none", "resting"]))
    if kind == "none":
        c.update(fields=rng.choice(["mixture", "layers"]), walls=rng.choice(["none", "none", "moving"]))
        if rng.random() < 0.3:
            c.update(psi=0, g_br=0.02)
        if rng.random() < 0.2:
            c["tau"] = 0.8
    c["domain_size"] = rng.random() < 0.3
    return _unnamed(c)


def _unnamed(c):
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs
def _noise(n, seed, k, amp):
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 4 + k)
    return amp * (2.0 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64) - 1.0)


def _system(case, dims, seed, rng):
    """Initial densities (torch, on the GPU), particles and walls of one system."""
    nx, ny, nz = dims
    N = nx * ny * nz
    amp = 0.01 if case["fields"] == "mixture" else 0.001
    if case["fields"] == "mixture":
        ra, rb = 0.7 + _noise(N, seed, 0, amp), 0.7 + _noise(N, seed, 1, amp)
    else:  # A below the middle plane, B above
        hi, lo = (1.4, 0.05) if case["fields"] == "lamellae" else (0.7, 0.04)
        below = torch.arange(N, device="cuda") // (nx * ny) < nz // 2
        ra = torch.where(below, hi, lo).double() + _noise(N, seed, 0, amp)
        rb = torch.where(below, lo, hi).double() + _noise(N, seed, 1, amp)
    kind = case["particles"]
    if kind == "none":
        radii, pos, quat, colour, dens = np.zeros((0, 2)), np.zeros((0, 3)), np.zeros((0, 4)), np.zeros(0), np.zeros(0)
    elif kind == "one":
        big = 0.5 * (min(dims) - 9)
        if case["systems"]:
            rperp = min(rng.uniform(3.0, 6.0), big)
            rpar = min(math.exp(rng.uniform(math.log(0.5), math.log(3.0))) * rperp, big)
            quat = tilt_quaternion(rng.uniform(0.0, 0.5 * math.pi), rng.uniform(0.0, 2.0 * math.pi))[None, :]
            colour = np.array([rng.uniform(-0.3, 0.3)])
        else:
            rpar, rperp = (12.0, 6.0) if case["fields"] == "lamellae" else (8.0, 4.0)
            rpar, rperp = min(rpar, big), min(rperp, big)
            quat, colour = shoemake_quaternions(rng, 1), np.zeros(1)
        radii, dens = np.array([[rpar, rperp]]), np.full(1, case["density"])
        pos = np.array([[nx / 2.0, ny / 2.0, nz / 2.0 - 0.5]]) + rng.uniform(-0.5, 0.5, (1, 3))
    else:
        # random sequential addition in one tile, repeated over the box
        rep = max(1, case["tile"])
        small = (nx // rep, ny // rep, nz // rep)
        if kind == "prolate":
            long, shape = 8.0, lambda r: (8.0, 4.0, 0.0)
        else:  # aspect ratio U[0.5, 2]
            long, shape = 5.0, lambda r: (4.0 * r.uniform(0.5, 2.0), 4.0, 0.0)
        count = max(1, round(case["phi"] * small[0] * small[1] * small[2] / (4.0 / 3.0 * math.pi * long * 16.0)))
        radii, pos, quat, colour = place_particles(small, rng, count, shape)
        shift = np.array([(i, j, k) for k in range(rep) for j in range(rep) for i in range(rep)], float) * np.array(small)
        pos = (pos[None] + shift[:, None]).reshape(-1, 3)
        radii, quat, colour = (np.tile(v, (len(shift),) + (1,) * (v.ndim - 1)) for v in (radii, quat, colour))
        if kind == "mixed":
            colour = rng.uniform(-0.3, 0.3, len(colour))
        dens = np.full(len(colour), case["density"])
    z = torch.arange(N, device="cuda") // (nx * ny)
    mask = None if case["walls"] == "none" else (z == 0) | (z == nz - 1)
    wall_u = (0.02, 0.005, 0.0) if case["walls"] == "moving" else None
    accel = (1e-5, 0.0, 0.0) if case["walls"] == "moving" else None
    return dict(dims=dims, ra=ra, rb=rb, radii=radii, pos=pos, quat=quat, colour=colour, dens=dens, mask=mask,
                wall_u=wall_u, accel=accel)


def _dims(case):
    if not case["systems"]:
        return [(case["nx"], case["ny"], case["nz"])]
    out, rng = [], np.random.default_rng(case["systems"])
    for _ in range(case["systems"]):
        nx, ny = (8 * int(rng.integers(4, 11)) for _ in range(2))
        out.append((nx, ny, 2 * nx + 8 * int(rng.integers(0, 5))))
    return out


def _systems(case, seed):
    rng = np.random.default_rng(int(seed))
    return [_system(case, d, int(seed) * 64 + k, rng) for k, d in enumerate(_dims(case))]


def prepare(case, seed):
    """The handle with its fields and particles, and the tensors the program records into."""
    systems = _systems(case, seed)
    args = [dict(dims=s["dims"], tau=case["tau"], g_br=case["g_br"], psi_kind=case["psi"],
                 max_particles=max(len(s["dens"]), 2 if case["pairs"] else 0),
                 max_radius=float(s["radii"].max()) if len(s["dens"]) else (1.0 if case["pairs"] else 0.0))
            for s in systems]
    if case["systems"]:
        handle = Batch(args, case["precision"])
        lats = list(handle.systems)
    else:
        handle = Lattice(precision=case["precision"], **args[0])
        lats = [handle]
    for lat, s in zip(lats, systems):
        if s["mask"] is not None:
            lat.set_static_solid(s["mask"].cpu().numpy(), s["wall_u"])
        lat.init_fields(s["ra"].cpu().numpy(), s["rb"].cpu().numpy())
        if len(s["dens"]):
            lat.add_ellipsoids(s["radii"], s["pos"], s["quat"], s["colour"], s["dens"])
        if s["accel"] is not None:
            lat.set_body_accel(s["accel"])
        if case["pairs"] and len(s["dens"]) > 1:
            lat.set_pair_interactions(True)
    if case["systems"]:
        handle.tune()
    N = sum(lat.N for lat in lats)
    f = lambda *shape, dtype=torch.float64: torch.empty(*shape, dtype=dtype, device="cuda")  # noqa: E731
    rec = dict(ra=f(N), rb=f(N), u=f(3 * N), own=f(N, dtype=torch.int32))
    return dict(case=case, handle=handle, lats=lats, rec=rec)


def run(state):
    """Some steps (with the health check that `step` makes), then the new state."""
    case, rec = state["case"], state["rec"]
    state["handle"].step(case["steps"])
    at = 0
    parts = []
    for lat in state["lats"]:
        end = at + lat.N
        lat.read_fields_dev(rec["ra"][at:end], rec["rb"][at:end], rec["u"][3 * at:3 * end], rec["own"][at:end])
        at = end
        if case["particles"] != "none":
            parts.append(lat.read_particles())
    dt = DTYPE[case["precision"]]
    out = {"rho_a": rec["ra"].to(dt), "rho_b": rec["rb"].to(dt), "u": rec["u"].to(dt), "owner": rec["own"]}
    if parts:
        p = {k: np.concatenate([q[k] for q in parts]) for k in parts[0]}
        for k in ("vel", "omega", "force", "torque"):
            p[k] = torch.from_numpy(p[k]).to(dt)
        out.update(p)
    if case["domain_size"]:
        out["domain_size"] = state["handle"].domain_size()
    return out


def work(case):
    """A pass reads and writes every population once a step; where tau = 1 the
    collision forgets all of a node but its two densities and its velocity,
    so these five numbers suffice. The record at the end is written once."""
    N = sum(a * b * c for a, b, c in _dims(case))
    s = STORE[case["precision"]]
    per = 2 * 5 * max(s, 4) if case["tau"] == 1.0 else 2 * 38 * s
    owner = 4 if case["particles"] != "none" or case["walls"] != "none" else 0
    read = 5 * 8 + 4 + (8 if case["domain_size"] else 0)
    return {"bytes": float(N * (case["steps"] * (per + owner) + read)), "flops": float(N * case["steps"] * 500)}


# ---------------------------------------------------------------- the time step in plain torch
_C = [(x, y, z) for z in (-1, 0, 1) for y in (-1, 0, 1) for x in (-1, 0, 1) if abs(x) + abs(y) + abs(z) <= 2]
_W = [{0: 1 / 3, 1: 1 / 18, 2: 1 / 36}[abs(x) + abs(y) + abs(z)] for x, y, z in _C]


def _from(a, c):
    """a(n - c) at n, for a field [z, y, x]."""
    return torch.roll(a, shifts=(c[2], c[1], c[0]), dims=(-3, -2, -1)) if any(c) else a


def _feq(k, rho, u):
    cu = sum(c * v for c, v in zip(_C[k], u) if c)
    return _W[k] * rho * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * (u[0] ** 2 + u[1] ** 2 + u[2] ** 2))


def _rot(q):
    w, x, y, z = q.T
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).reshape(-1, 3, 3)


class _Plain:
    def __init__(self, case, s):
        t = lambda v: torch.as_tensor(v, dtype=torch.float64, device="cuda")  # noqa: E731
        self.case, self.nxyz = case, s["dims"]
        self.shape = s["dims"][::-1]
        self.L = t(s["dims"])
        self.rho0 = [float(s["ra"].mean()), float(s["rb"].mean())]
        self.accel = s["accel"] or (0.0, 0.0, 0.0)
        self.wall_u = t(s["wall_u"] or (0.0, 0.0, 0.0))
        self.radii, self.X, self.q = t(s["radii"]), t(s["pos"]) % self.L, t(s["quat"])
        self.q = self.q / self.q.norm(dim=1, keepdim=True)
        self.colour, n = t(s["colour"]), len(s["dens"])
        rp, ro = self.radii.T
        self.M = t(s["dens"]) * 4 / 3 * math.pi * rp * ro ** 2
        i_o, i_p = self.M * (ro ** 2 + rp ** 2) / 5, self.M * 2 * ro ** 2 / 5
        self.I = torch.stack([i_o, i_o, i_p], 1)
        z = lambda: torch.zeros(n, 3, dtype=torch.float64, device="cuda")  # noqa: E731
        self.V, self.W, self.Lm, self.J, self.H = z(), z(), z(), z(), z()
        self.F, self.T = z(), z()
        self.wall = None if s["mask"] is None else s["mask"].reshape(self.shape)
        self.own = self.raster()
        fluid = self.own == -1
        zero = torch.zeros((), dtype=torch.float64, device="cuda")
        rho = [s["ra"].reshape(self.shape), s["rb"].reshape(self.shape)]
        self.f = [torch.stack([torch.where(fluid, _W[k] * r, zero) for k in range(19)]) for r in rho]

    def raster(self):
        n = len(self.M)
        far = 2 ** 30
        own = torch.full((int(self.L.prod()),), far, dtype=torch.int64, device="cuda")
        if n:
            rb = int(math.ceil(float(self.radii.max()))) + 1
            g = torch.arange(-rb, rb + 1, device="cuda")
            off = torch.stack(torch.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
            R, L = _rot(self.q), self.L.long()
            for a in range(0, n, 1024):
                p = torch.arange(a, min(a + 1024, n), device="cuda")
                node = torch.floor(self.X[p]).long()[:, None] + off
                d = (node - self.X[p][:, None]) @ R[p]
                ro, rp = self.radii[p, 1][:, None], self.radii[p, 0][:, None]
                inside = (d[..., 0] ** 2 + d[..., 1] ** 2) / ro ** 2 + d[..., 2] ** 2 / rp ** 2 <= 1
                node = node % L
                idx = (node[..., 0] + L[0] * (node[..., 1] + L[1] * node[..., 2]))[inside]
                own.scatter_reduce_(0, idx, p[:, None].expand_as(inside)[inside], "amin")
        own = torch.where(own == far, -1, own).reshape(self.shape)
        return own if self.wall is None else torch.where(self.wall, -2, own)

    def psi(self, rho):
        return rho if self.case["psi"] == 0 else -torch.expm1(-rho)

    def arm(self, node, p):
        """Minimum-image offset of nodes (z, y, x) from the centres of particles p."""
        d = torch.stack([node[2], node[1], node[0]], 1).double() - self.X[p]
        return d - self.L * torch.round(d / self.L)

    def step(self):
        case, tau = self.case, self.case["tau"]
        fluid = self.own == -1
        solid = ~fluid
        zero = torch.zeros((), dtype=torch.float64, device="cuda")
        rho = [f.sum(0) for f in self.f]
        # shell nodes take the mean density of their fluid neighbours (Eq. (10))
        psi = []
        any_solid = bool(solid.any())
        if any_solid:
            links = sum(_from(fluid.double(), c) for c in _C if any(c))
        for k in range(2):
            p = self.psi(rho[k])
            if any_solid:
                mean = sum(_from(rho[k], c) for c in _C if any(c)) / links.clamp(min=1)
                if len(self.M):
                    tint = (self.colour.clamp(min=0) if k == 0 else (-self.colour).clamp(min=0))
                    mean = mean + torch.where(self.own >= 0, tint[self.own.clamp(min=0)], zero)
                p = torch.where(solid, torch.where(links > 0, self.psi(mean), zero), p)
            psi.append(p)
        S = [[sum(c[d] * _from(p, tuple(-v for v in c)) for c in _C if c[d]) for d in range(3)] for p in psi]
        rt = torch.where(fluid, rho[0] + rho[1], torch.ones_like(rho[0]))
        u = [sum(c[d] * (self.f[0][k] + self.f[1][k]) for k, c in enumerate(_C) if c[d]) / rt for d in range(3)]
        post = []
        for k in range(2):
            r = torch.where(fluid, rho[k], torch.ones_like(rho[k]))
            ratio = -case["g_br"] * torch.where(r == 0, torch.ones_like(r), self.psi(r) / r)
            uk = [u[d] + tau * (ratio * S[1 - k][d] + self.accel[d]) for d in range(3)]
            post.append(torch.stack([torch.where(fluid, self.f[k][i] - (self.f[k][i] - _feq(i, r, uk)) / tau, zero)
                                     for i in range(19)]))
        # streaming with moving bounce-back (Eq. (4)) and the links' force (Eq. (5))
        self.F.zero_()
        self.T.zero_()
        new = [torch.empty_like(f) for f in self.f]
        for i, c in enumerate(_C):
            back = _C.index(tuple(-v for v in c))
            came = [_from(p[i], c) for p in post]
            if any(c) and any_solid:
                hit = fluid & _from(solid, c)
                node = torch.nonzero(hit, as_tuple=True)
                who = _from(self.own, c)[hit]
                cv = torch.tensor(c, dtype=torch.float64, device="cuda")
                ub = self.wall_u.expand(len(who), 3).clone()
                body = who >= 0
                r = None
                if len(self.M):
                    p = who.clamp(min=0)
                    r = self.arm(node, p)
                    ub = torch.where(body[:, None], self.V[p] + torch.cross(self.W[p], r, dim=1), ub)
                push = zero
                for k in range(2):
                    out = post[k][back][hit]
                    C = 6 * _W[i] * rho[k][hit] * (ub @ cv)
                    came[k][hit] = out + C
                    push = push + 2 * out + C
                if r is not None:
                    dF = push[:, None] * -cv
                    self.F.index_add_(0, p[body], dF[body])
                    self.T.index_add_(0, p[body], torch.cross(r, dF, dim=1)[body])
            for k in range(2):
                new[k][i] = torch.where(fluid, came[k], zero)
        self.f = new
        if len(self.M):
            self.bodies()
            self.move(fluid)

    def bodies(self):
        if self.case["pairs"] and len(self.M) > 1:
            dF, dT = self.pair_terms()
            self.F += dF
            self.T += dT
        self.F += self.J
        self.T += self.H
        self.J.zero_()
        self.H.zero_()
        self.V = self.V + self.F / self.M[:, None]
        self.X = (self.X + self.V) % self.L
        self.Lm = self.Lm + self.T
        R = _rot(self.q)
        self.W = (R @ ((R.transpose(1, 2) @ self.Lm[:, :, None])[..., 0] / self.I)[:, :, None])[..., 0]
        th = self.W.norm(dim=1, keepdim=True)
        v = self.W * torch.where(th < 1e-12, 0.5, torch.sin(0.5 * th) / th.clamp(min=1e-300))
        w, s, qv = torch.cos(0.5 * th), self.q[:, :1], self.q[:, 1:]
        q = torch.cat([w * s - (v * qv).sum(1, keepdim=True), w * qv + s * v + torch.cross(v, qv, dim=1)], 1)
        self.q = q / q.norm(dim=1, keepdim=True)

    def move(self, before):
        """Nodes that change side: kill gives the node's momentum to the particle, fill takes it (about the new centre)."""
        old, self.own = self.own, self.raster()
        now = self.own == -1
        both = before & now
        rho = [f.sum(0) for f in self.f]
        zero = torch.zeros((), dtype=torch.float64, device="cuda")
        kill, fill = before & ~now, (old >= 0) & now
        if bool(kill.any()):
            node, p = torch.nonzero(kill, as_tuple=True), self.own[kill]
            j = torch.stack([sum(c[d] * (self.f[0][k] + self.f[1][k])[kill] for k, c in enumerate(_C) if c[d]) for d in range(3)], 1)
            self.J.index_add_(0, p, j)
            self.H.index_add_(0, p, torch.cross(self.arm(node, p), j, dim=1))
        if bool(fill.any()):
            node, p = torch.nonzero(fill, as_tuple=True), old[fill]
            r = self.arm(node, p)
            ub = self.V[p] + torch.cross(self.W[p], r, dim=1)
            links = sum(_from(both.double(), c)[fill] for c in _C if any(c))
            total = zero
            for k in range(2):
                mean = sum(_from(torch.where(both, rho[k], zero), c)[fill] for c in _C if any(c)) / links.clamp(min=1)
                mean = torch.where(links > 0, mean, self.rho0[k])
                total = total + mean
                for i in range(19):
                    self.f[k][i][fill] = _feq(i, mean, list(ub.T))
            j = total[:, None] * ub
            self.J.index_add_(0, p, -j)
            self.H.index_add_(0, p, -torch.cross(r, j, dim=1))
        for k in range(2):
            self.f[k] = torch.where(now, self.f[k], zero)

    def pair_terms(self, K_H=100.0, gap=2.0 / 3.0):
        """Hertz / Berne-Pechukas and lubrication (Eqs. (6)-(9)), forces as gradients of the energy."""
        X = self.X.clone().requires_grad_(True)
        o = _rot(self.q)[:, :, 2].clone().requires_grad_(True)
        d = self.X[:, None] - self.X[None]
        d = d - self.L * torch.round(d / self.L)
        near = 2 * float(self.radii.max()) + gap
        i, j = torch.nonzero(torch.triu(d.norm(dim=2) < near, diagonal=1), as_tuple=True)
        rp, ro = (0.5 * (self.radii[i] + self.radii[j])).T
        r = X[i] - X[j]
        r = r - self.L * torch.round(r.detach() / self.L)
        rn = r.norm(dim=1)
        e = r / rn[:, None]
        chi = (rp ** 2 - ro ** 2) / (rp ** 2 + ro ** 2)
        a, b, c = (e * o[i]).sum(1), (e * o[j]).sum(1), (o[i] * o[j]).sum(1)
        G = (a + b) ** 2 / (1 + chi * c) + (a - b) ** 2 / (1 - chi * c)
        sig = 2 * ro / torch.sqrt(1 - 0.5 * chi * G)
        eps = K_H * (2 * ro) ** 2.5 / torch.sqrt(1 - (chi * c) ** 2)
        x = rn / sig
        reach = rn < 2 * torch.maximum(rp, ro) + gap
        energy = torch.where(reach & (x < 1), eps * (1 - x).clamp(min=1e-300) ** 2.5, torch.zeros_like(x)).sum()
        gX, go = torch.autograd.grad(energy, (X, o), allow_unused=True)
        F, T = -gX, -torch.cross(o.detach(), go, dim=1)
        e, rn, sig = e.detach(), rn.detach(), sig.detach()
        h = rn - sig
        mu = (self.rho0[0] + self.rho0[1]) * (self.case["tau"] - 0.5) / 3
        un = (e * (self.V[i] - self.V[j])).sum(1)
        mag = -1.5 * math.pi * mu * (0.5 * sig) ** 2 * un * (1 / h.clamp(min=0.25 * gap) - 1 / gap)
        lub = torch.where((reach & (h < gap))[:, None], mag[:, None] * e, torch.zeros_like(e))
        F = F.index_add(0, i, lub).index_add(0, j, -lub)
        return F, T

    def state(self):
        rho = [f.sum(0).reshape(-1) for f in self.f]
        rt = rho[0] + rho[1]
        u = torch.stack([sum(c[d] * (self.f[0][k] + self.f[1][k]) for k, c in enumerate(_C) if c[d]).reshape(-1)
                         for d in range(3)], 1) / torch.where(rt == 0, torch.ones_like(rt), rt)[:, None]
        return rho[0], rho[1], u.reshape(-1)

    def sizes(self):
        """Lateral domain sizes (Eq. (12)) of rho_A - rho_B."""
        phi = self.f[0].sum(0) - self.f[1].sum(0)
        S = torch.fft.fftn(phi - phi.mean()).abs() ** 2 / phi.numel()
        S[0, 0, 0] = 0
        k2 = []
        for d in range(3):
            n = self.nxyz[d]
            k = 2 * math.pi * torch.fft.fftfreq(n, dtype=torch.float64, device="cuda")
            k2.append(float((S.sum(dim=[a for a in range(3) if a != 2 - d]) * k ** 2).sum() / S.sum()))
        L = [2 * math.pi / math.sqrt(v) if v > 0 else math.inf for v in k2]
        return np.array(L + [sum(L) / 3] + k2 + [float(S.sum())])


def exact(case, seed):
    """What `run` returns after its first pass on a new state, in double. The
    largest boxes would take minutes and are left out."""
    if not case["systems"] and case["nx"] * case["ny"] * case["nz"] * case["steps"] > 8e8:
        return None
    sims = []
    with torch.no_grad():
        for s in _systems(case, seed):
            p = _Plain(case, s)
            for _ in range(case["steps"]):
                with torch.enable_grad() if case["pairs"] else torch.no_grad():
                    p.step()
            sims.append(p)
        parts = [p.state() for p in sims]
        out = {"rho_a": torch.cat([v[0] for v in parts]), "rho_b": torch.cat([v[1] for v in parts]),
               "u": torch.cat([v[2] for v in parts]), "owner": None}
        if case["particles"] != "none":
            for k, name in (("X", "pos"), ("q", "quat"), ("V", "vel"), ("W", "omega"), ("F", "force"), ("T", "torque")):
                out[name] = torch.cat([getattr(p, k) for p in sims]).cpu()
        if case["domain_size"]:
            out["domain_size"] = sims[0].sizes()
    return out
