"""The FP64 step at tau = 1, which carries densities and velocity instead of
populations, against the oracle at the edges of its columns (32 x 8 nodes) and
of their runs along z: boxes narrower than a column, one node past it, the
smallest box; without particles, with nodes that touch one, two and several
bodies, with walls and a body force. Each run saves its state half way and
goes on from the image in a second handle (populations formed from the moments
and summed again): both must end bit for bit alike. Tolerances: those of the
FP64 parity tests."""
import numpy as np
import pytest

from paper_1109_3277_amd import workloads as W
from tests.parity_util import check, compare, log

pytestmark = pytest.mark.gpu


def _cluster(dims, seed):
    """Spheres around one node of a small box, so that nodes touch several bodies."""
    ra, rb = W.uniform_fields(dims, seed, 0.7, 0.7, 0.01)
    c = np.array(dims) / 2.0
    off = 3.2 * np.array([[1, 0, 0], [-1, 0, 0], [0, 1, 0], [0, -1, 0], [0, 0, 1], [0, 0, -1]])
    n = len(off)
    rng = np.random.default_rng(seed)
    return W.System("cluster", dims, 1.0, 0.08, ra, rb, np.full((n, 2), 2.4), c + off + rng.uniform(-0.1, 0.1, (n, 3)),
                    W.shoemake_quaternions(rng, n), rng.uniform(-0.2, 0.2, n), np.full(n, 8.0), seed=seed)


CASES = {
    "smallest": lambda: (W.spinodal_system(dims=(3, 3, 3), seed=1), False),
    "narrow": lambda: (W.spinodal_system(dims=(31, 7, 4), seed=2), False),
    "past-the-column": lambda: (W.spinodal_system(dims=(33, 9, 67), seed=3), False),
    "particles": lambda: (W.bijel_system(dims=(33, 25, 41), seed=4, phi=0.12, rpar=5.0, rperp=3.0), False),
    "several-bodies": lambda: (_cluster((20, 17, 19), 5), False),
    "walls": lambda: (W.interface_system(dims=(34, 18, 35), rpar=5.0, rperp=3.0, delta_rho=0.1, seed=6), True),
    "walls-no-particle": lambda: (W.spinodal_system(dims=(35, 10, 9), seed=7), True),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_moment_step_fp64(name):
    import oracle
    from paper_1109_3277_amd.binding import Lattice

    s, walls = CASES[name]()
    log(f"case {name} dims={s.dims} np={s.n_particles}")
    mask = W.wall_mask(s.dims) if walls else None
    wall_u, accel = (0.01, -0.005, 0.0), (1e-5, 2e-6, 0.0)

    def handle():
        g = Lattice(s.dims, 1.0, s.g_br, s.psi_kind, "fp64", max_particles=s.n_particles, max_radius=s.max_radius)
        if walls:
            g.set_static_solid(mask, wall_u)
        return g

    def start(x):
        x.init_fields(s.rho_a, s.rho_b)
        if s.n_particles:
            x.add_ellipsoids(s.radii, s.pos, s.quat, s.delta_rho, s.density)
        if walls:
            (x.set_body_accel if isinstance(x, Lattice) else x.set_accel)(accel)

    o = oracle.Oracle(s.dims, 1.0, s.g_br, s.psi_kind)
    if walls:
        o.set_walls(mask, np.tile(wall_u, (s.N, 1)))
    start(o)
    o.step(40)
    a = handle()
    start(a)
    a.step(20)
    image = a.save_state()
    a.step(20)
    res = compare(o, a, s.dims, s.radii)
    log(f"  {res}")
    check(res, 1e-12, vel_gate=1e-10, particles=s.n_particles > 0)
    b = handle()
    b.load_state(image)
    if walls:
        b.set_body_accel(accel)
    b.step(20)
    for u, v in zip(a.read_fields(), b.read_fields()):
        assert np.array_equal(u, v)
    pa, pb = a.read_particles(), b.read_particles()
    for k in pa:
        assert np.array_equal(pa[k], pb[k]), k


def test_moment_step_matches_populations():
    """tau one ulp above 1 takes the general path: the two paths agree to rounding."""
    from paper_1109_3277_amd.binding import Lattice

    s = W.bijel_system(dims=(40, 40, 40), seed=8, phi=0.12, rpar=6.0, rperp=3.0)
    out = []
    for tau in (1.0, float(np.nextafter(1.0, 2.0))):
        g = Lattice(s.dims, tau, s.g_br, s.psi_kind, "fp64", max_particles=s.n_particles, max_radius=s.max_radius)
        g.init_fields(s.rho_a, s.rho_b)
        g.add_ellipsoids(s.radii, s.pos, s.quat, s.delta_rho, s.density)
        g.step(60)
        out.append((g.read_fields(), g.stats()))
    (fa, sa), (fb, sb) = out
    assert np.array_equal(fa[3], fb[3])
    for k in range(2):
        assert np.abs(fa[k] - fb[k]).max() <= 1e-12 * np.abs(fb[k]).max()
    assert np.abs(fa[2] - fb[2]).max() <= 1e-10 * max(np.abs(fb[2]).max(), 1e-3)
    assert np.allclose(sa, sb, rtol=1e-11, atol=1e-9)
