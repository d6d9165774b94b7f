"""Particle passes shared by several blocks: the number of blocks per particle
follows from the particle count (16 up to 64 particles, one from 513 on). At its
edges, and for one ellipsoid nearly as wide as its box, with bodies that cross
nodes; a batch of the same systems bit for bit alike. Against the oracle at the
gates of the parity tests."""
import numpy as np
import pytest

from paper_1109_3277_amd import workloads as W
from tests.parity_util import check, compare, log, run_oracle

pytestmark = pytest.mark.gpu


def _lattice_of(count, seed):
    """count small ellipsoids on a cubic lattice, drifting with the fluid."""
    per = 9 if count > 64 else 5
    h = 6.0
    side = int(per * h)
    dims = (side, side, side)
    rng = np.random.default_rng(seed)
    pos = np.array([[x, y, z] for z in range(per) for y in range(per) for x in range(per)], float)[:count] * h
    ra, rb = W.uniform_fields(dims, seed, 0.7, 0.7, 0.01)
    return W.System("shares", dims, 1.0, 0.08, ra, rb, np.tile([2.3, 1.7], (count, 1)),
                    pos + rng.uniform(-0.4, 0.4, pos.shape), W.shoemake_quaternions(rng, count),
                    rng.uniform(-0.1, 0.1, count), np.full(count, 8.0), seed=seed)


def _cases():
    out = {f"np{n}": _lattice_of(n, n) for n in (64, 65, 512, 513)}
    out["wide"] = W.interface_system(dims=(24, 25, 26), rpar=11.9, rperp=7.0, delta_rho=0.1, seed=3)
    return out


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_particle_shares(precision):
    from paper_1109_3277_amd.binding import Batch, Lattice

    cases = _cases()
    batch = Batch([{"dims": s.dims, "tau": s.tau, "g_br": s.g_br, "psi_kind": s.psi_kind,
                    "max_particles": s.n_particles, "max_radius": s.max_radius} for s in cases.values()], precision)
    drift = (0.03, -0.02, 0.025)

    def start(x, s):
        x.init_fields(s.rho_a, s.rho_b)
        x.add_ellipsoids(s.radii, s.pos, s.quat, s.delta_rho, s.density)
        for k in range(s.n_particles):
            x.set_particle_motion(k, vel=drift)

    for k, s in enumerate(cases.values()):
        start(batch[k], s)
    batch.step(12)
    for k, (name, s) in enumerate(cases.items()):
        g = Lattice(s.dims, s.tau, s.g_br, s.psi_kind, precision, max_particles=s.n_particles, max_radius=s.max_radius)
        start(g, s)
        g.step(12)
        for u, v in zip(g.read_fields(), batch[k].read_fields()):
            assert np.array_equal(u, v), name
        pa, pb = g.read_particles(), batch[k].read_particles()
        assert all(np.array_equal(pa[q], pb[q]) for q in pa), name
        o = run_oracle(s, 0)
        for q in range(s.n_particles):
            o.set_particle_motion(q, V=drift)
        o.step(12)
        res = compare(o, g, s.dims, s.radii)
        log(f"case shares {name} {precision}: {res}")
        if precision == "fp64":
            check(res, 1e-12, vel_gate=1e-10)
        else:
            check(res, 1e-5)
        g.close()
    batch.close()
