"""Steps of a lone handle recorded by its caller into a HIP graph
(lb_step_async, "for timing and graph capture by the caller"): two steps
captured right after the fields are set, or after steps were run, and replayed
several times with readouts, saves, loads and new fields in between. Every state
must be bit for bit the one that the same steps give when they are called."""
import hashlib

import numpy as np
import pytest

from paper_1109_3277_amd import workloads as W
from tests.parity_util import log

pytestmark = pytest.mark.gpu


def _system(kind, tau):
    if kind == "particles":
        s = W.bijel_system(dims=(33, 25, 41), seed=4, phi=0.12, rpar=5.0, rperp=3.0)
    elif kind == "walls":
        s = W.spinodal_system(dims=(35, 10, 9), seed=7)
    else:
        s = W.spinodal_system(dims=(33, 9, 20), seed=3)
    s.tau = tau
    return s


def _handle(s, kind, prec):
    from paper_1109_3277_amd.binding import Lattice

    g = Lattice(s.dims, s.tau, s.g_br, s.psi_kind, prec, max_particles=s.n_particles, max_radius=s.max_radius)
    if kind == "walls":
        g.set_static_solid(W.wall_mask(s.dims), (0.01, -0.005, 0.0))
    g.init_fields(s.rho_a, s.rho_b)
    if s.n_particles:
        g.add_ellipsoids(s.radii, s.pos, s.quat, s.delta_rho, s.density)
    return g


def _digest(image):
    return hashlib.sha256(image).hexdigest()  # (a failed comparison of images themselves prints for minutes)


def _image(g):
    return _digest(g.save_state())


def _same(a, b, what):
    for k, (x, y) in enumerate(zip(a.read_fields(), b.read_fields())):
        assert np.array_equal(x, y), (what, "field", k)
    pa, pb = a.read_particles(), b.read_particles()
    for k in pa:
        assert np.array_equal(pa[k], pb[k]), (what, k)
    assert np.array_equal(a.stats(), b.stats()), (what, "stats")


@pytest.mark.parametrize("warm", [0, 3])
@pytest.mark.parametrize("kind", ["plain", "walls", "particles"])
@pytest.mark.parametrize("prec,tau", [("fp64", 1.0), ("fp64", 1.25), ("fp32", 1.0)])
def test_captured_steps_replay(kind, prec, tau, warm):
    import torch

    if tau != 1.0 or prec != "fp64":
        # a population run that has stepped starts from the densities of its last
        # step: a graph recorded then holds no density pass of its own and goes on
        # from new fields only where there are no particles
        if warm and kind == "particles":
            pytest.skip("populations: recorded after steps, particles present")
    s = _system(kind, tau)
    log(f"case {kind} {prec} tau={tau} warm={warm} dims={s.dims} np={s.n_particles}")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        a, b = _handle(s, kind, prec), _handle(s, kind, prec)
        if warm:
            a.step(warm)
            b.step(warm)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            a.step_async(2)
        _same(a, b, "captured, not run")
        assert _image(a) == _image(b)
        images = []
        for r in range(3):
            graph.replay()
            b.step(2)
            _same(a, b, f"replay {r}")
            images.append(a.save_state())
            assert _digest(images[r]) == _image(b), f"image after replay {r}"
        # new fields (a flow; the same mean densities, which the kernels take as
        # arguments) under the same particles
        for x in (a, b):
            x.init_fields(s.rho_a, s.rho_b, np.tile([0.01, -0.02, 0.005], (s.N, 1)))
        _same(a, b, "new fields")
        assert _image(a) == _image(b)
        for r in range(2):
            graph.replay()
            b.step(2)
            _same(a, b, f"new fields, replay {r}")
        # back to the first image; a readout only after the replays
        for x in (a, b):
            x.load_state(images[0])
        graph.replay()
        graph.replay()
        b.step(4)
        _same(a, b, "loaded")
        assert _image(a) == _image(b) == _digest(images[2])
        a.close()
        b.close()
