"""The FP64 step in populations (tau != 1; tau = 1 steps in moments) where its
kernels change path: z-runs of ragged tiles, nodes that link to three and to five
particles, the row kernel's widths, particles placed mid-run, and checkpoints
(plain form, bounce masks). Against the oracle at the gates of the FP64 parity
tests (densities 1e-12, particle velocities 1e-10)."""
import numpy as np
import pytest

from paper_1109_3277_amd import workloads as W
from tests.parity_util import check, compare, log, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

TAUS = [0.8, 1.25]


def _parity(s, steps):
    log(f"case {s.name} dims={s.dims} np={s.n_particles} tau={s.tau} steps={steps}")
    o, g = run_oracle(s, steps), run_gpu(s, steps, "fp64")
    res = compare(o, g, s.dims, s.radii)
    check(res, 1e-12, vel_gate=1e-10)
    assert res["e_mass"] <= 1e-12, res
    g.close()


@pytest.mark.parametrize("tau", TAUS)
def test_z_runs_of_ragged_tiles(tau):
    _parity(W.bijel_system(dims=(70, 516, 12), seed=21, phi=0.1, rpar=4.5, rperp=2.5, tau=tau), 30)


@pytest.mark.parametrize("tau", TAUS)
@pytest.mark.parametrize("bodies", [1, 2, 3, 5])
def test_node_that_links_to_several_particles(bodies, tau):
    """Spheres around node (12, 12, 12): it links to each of them (asserted)."""
    import oracle

    dims = (24, 24, 24)
    ra, rb = W.uniform_fields(dims, 23, 0.7, 0.7, 0.01)
    pos = np.array([[9.0, 12.0, 12.0], [15.0, 12.0, 12.0], [12.0, 15.0, 12.0], [12.0, 9.0, 12.0],
                    [12.0, 12.0, 15.0]])[:bodies]
    s = W.System(f"bodies{bodies}", dims, tau, 0.08, ra, rb, np.full((bodies, 2), 2.4), pos,
                 np.tile([1.0, 0, 0, 0], (bodies, 1)), np.array([0.05, -0.05, 0.0, 0.03, -0.02])[:bodies],
                 np.full(bodies, 10.0))
    o = oracle.Oracle(dims, tau, 0.08)
    o.init_fields(ra, rb)
    o.add_ellipsoids(s.radii, s.pos, s.quat, s.delta_rho, s.density)
    own = o.owner().reshape(24, 24, 24)
    near = [own[12, 12, 11], own[12, 12, 13], own[12, 13, 12], own[12, 11, 12], own[13, 12, 12]]
    assert own[12, 12, 12] == -1 and near[:bodies] == list(range(bodies))
    _parity(s, 20)


@pytest.mark.parametrize("tau", TAUS)
@pytest.mark.parametrize("dims", [(64, 8, 5), (64, 16, 12), (128, 6, 5), (128, 16, 12), (256, 4, 5)])
def test_rows_without_solids(dims, tau):
    """64 and 128 nodes: the row kernel (aligned stores, wave edges, periodic
    seam); 256: tiles."""
    ra, rb = W.uniform_fields(dims, 30 + dims[0], 0.7, 0.7, 0.01)
    s = W.System(f"rows{dims}", dims, tau, 0.08, ra, rb)
    log(f"case {s.name} tau={tau}")
    o, g = run_oracle(s, 40), run_gpu(s, 40, "fp64")
    check(compare(o, g, dims), 1e-12, particles=False)
    g.close()


@pytest.mark.parametrize("tau", TAUS)
def test_particles_placed_mid_run(tau):
    import oracle
    from paper_1109_3277_amd.binding import Lattice

    s = W.bijel_system(dims=(40, 40, 40), seed=29, phi=0.1, tau=tau)
    h = s.n_particles // 2
    log(f"case placed mid-run np={h}+{s.n_particles - h} tau={tau}")
    o = oracle.Oracle(s.dims, tau, s.g_br)
    g = Lattice(s.dims, tau, s.g_br, max_particles=s.n_particles, max_radius=s.max_radius)
    for x in (o, g):
        x.init_fields(s.rho_a, s.rho_b)
        x.add_ellipsoids(s.radii[:h], s.pos[:h], s.quat[:h], s.delta_rho[:h], s.density[:h])
        x.step(30)
        x.add_ellipsoids(s.radii[h:], s.pos[h:], s.quat[h:], s.delta_rho[h:], s.density[h:])
        x.step(30)
    check(compare(o, g, s.dims, s.radii), 1e-12, vel_gate=1e-10)
    g.close()


@pytest.mark.parametrize("tau", TAUS)
def test_checkpoint_in_populations(tau):
    """A saved run goes on as one that was not saved, and as one that was loaded,
    bit for bit."""
    from paper_1109_3277_amd.binding import Lattice

    s = W.bijel_system(dims=(32, 32, 32), seed=23, phi=0.12, tau=tau)
    log(f"case checkpoint np={s.n_particles} tau={tau}")
    a = run_gpu(s, 25, "fp64")
    image = a.save_state()
    a.step(25)
    b = run_gpu(s, 50, "fp64")
    c = Lattice(s.dims, tau, s.g_br, s.psi_kind, "fp64", max_particles=s.n_particles, max_radius=s.max_radius)
    c.load_state(image)
    c.step(25)
    for x in (b, c):
        for u, v in zip(a.read_fields(), x.read_fields()):
            assert np.array_equal(u, v)
        pa, px = a.read_particles(), x.read_particles()
        for k in pa:
            assert np.array_equal(pa[k], px[k]), k
