"""The two ways the particle-particle pass finds its pairs, at the counts where
they and their 64-wide rounds change: two particles, one more than a wave, and
2048 / 2049, the last all-pairs count and the first with the cell list, with
contacts across the periodic seams. Against the oracle at the FP64 gates of the
parity tests."""
import numpy as np
import pytest

from paper_1109_3277_amd.workloads import System, shoemake_quaternions, uniform_fields
from tests.parity_util import check, compare, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [2, 65, 2048, 2049])
def test_pair_paths_fp64(count):
    import oracle
    from paper_1109_3277_amd.binding import Lattice

    per = 13 if count > 1000 else 5
    side = 64 if count > 1000 else 25
    dims, h = (side, side, side), side / per  # spacing 4.92 or 5: inside 2 R + 2/3
    rng = np.random.default_rng(count)
    pos = np.array([[x, y, z] for z in range(per) for y in range(per) for x in range(per)], float)[:count] * h
    pos = pos + rng.uniform(-0.15, 0.15, pos.shape)
    ra, rb = uniform_fields(dims, count, 0.7, 0.7, 0.01)
    s = System("pair-paths", dims, 1.0, 0.08, ra, rb, np.tile([2.4, 2.1], (count, 1)), pos,
               shoemake_quaternions(rng, count), np.zeros(count), np.full(count, 10.0))
    u = 0.02 * rng.uniform(-1, 1, (s.N, 3))
    o = oracle.Oracle(s.dims, s.tau, s.g_br, s.psi_kind)
    g = Lattice(s.dims, s.tau, s.g_br, s.psi_kind, "fp64", max_particles=count, max_radius=s.max_radius)
    for x in (o, g):
        x.init_fields(s.rho_a, s.rho_b, u)
        x.add_ellipsoids(s.radii, s.pos, s.quat, s.delta_rho, s.density)
    o.set_pairs(True, 100.0, 2.0 / 3.0)
    g.set_pair_interactions(True, 100.0, 2.0 / 3.0)
    o.step(8)
    g.step(8)
    res = compare(o, g, s.dims, s.radii)
    log(f"case pair-paths np={count}: {res}")
    check(res, 1e-12, vel_gate=1e-10)
