"""The launch that fills particle shells and wall nodes and clears the next owner
copy: walls with no, few (shared by blocks) and many drifting ellipsoids, kept
densities and Psi = rho. Against the oracle at the gates of the parity tests."""
import numpy as np
import pytest

from paper_1109_3277_amd import workloads as W
from tests.parity_util import check, compare, log

pytestmark = pytest.mark.gpu

DRIFT = (0.03, -0.02, 0.01)


@pytest.mark.parametrize("precision,tau", [("fp64", 1.0), ("fp64", 1.25), ("fp32", 1.0)])
@pytest.mark.parametrize("count,psi_kind", [(0, 1), (5, 0), (5, 1), (513, 1)])
def test_walls_and_particles(count, psi_kind, precision, tau):
    import oracle
    from paper_1109_3277_amd.binding import Lattice

    side = 7 if count > 5 else 3
    nz = 11 if count > 5 else 3
    dims = (7 * side, 7 * side, 7 * nz + 2)
    N = int(np.prod(dims))
    z = np.arange(N) // (dims[0] * dims[1])
    walls = (z == 0) | (z == dims[2] - 1)
    rng = np.random.default_rng(count)
    grid = [(x, y, w) for w in range(nz) for y in range(side) for x in range(side)]
    pos = (np.array(grid, float)[:count].reshape(-1, 3) + 0.5) * 7.0 + (0.0, 0.0, 1.0)
    ra, rb = W.uniform_fields(dims, count + 1, 0.7, 0.7, 0.01)
    radii = np.tile([2.3, 1.7], (count, 1))
    o = oracle.Oracle(dims, tau, 0.08, psi_kind)
    g = Lattice(dims, tau, 0.08, psi_kind, precision, max_particles=count, max_radius=2.3 if count else 0.0)
    o.set_walls(walls, np.tile(np.array([0.01, -0.004, 0.0]), (N, 1)))
    g.set_static_solid(walls, [0.01, -0.004, 0.0])
    for x in (o, g):
        x.init_fields(ra, rb)
        if count:
            x.add_ellipsoids(radii, pos, W.shoemake_quaternions(np.random.default_rng(7), count),
                             np.linspace(-0.1, 0.1, count), np.full(count, 8.0))
    for q in range(count):
        o.set_particle_motion(q, V=DRIFT)
        g.set_particle_motion(q, vel=DRIFT)
    o.step(15)
    g.step(15)
    res = compare(o, g, dims, radii if count else None)
    log(f"case walls np={count} psi={psi_kind} {precision} tau={tau}: {res}")
    if precision == "fp64":
        check(res, 1e-12, vel_gate=1e-10)
    else:
        check(res, 1e-5)
    g.close()
