"""Checkpoints of the FP64 step at tau = 1, whose populations are formed from
the state one step before: right after the fields were set, after particles were
placed (before any step and mid-run), and after the body force changed. A loaded
image gives the same image again, and the run that goes on from it ends bit for
bit where the saved run ends."""
import hashlib

import numpy as np
import pytest

from paper_1109_3277_amd import workloads as W
from tests.parity_util import log

pytestmark = pytest.mark.gpu

def _digest(image):
    return hashlib.sha256(image).hexdigest()  # (a failed comparison of images themselves prints for minutes)


# what is done to a handle before it is saved: numbers are steps
STORIES = {
    "fresh": ["init"],
    "fresh-then-particles": ["init", "add0"],
    "first-steps-then-particles": ["init", 7, "add0"],
    "particles-then-more": ["init", "add0", 6, "add1"],
    "particles-one-step-then-more": ["init", "add0", 1, "add1"],
    "force-changed": ["init", "add0", "force0", 5, "force1"],
    "force-changed-no-particles": ["init", "force0", 4, "force1"],
    "particles-and-force": ["init", "force0", 5, "add0", "force1", 3, "add1", "force0"],
    "saved-twice": ["init", "add0", 5, "save", 4],
    "fields-set-again": ["init", "add0", 5, "init", 3],
    "loaded-then-particles": ["init", "add0", 5, "reload", "add1"],
}
FORCES = {"force0": (1e-5, 2e-6, 0.0), "force1": (-4e-5, 0.0, 3e-5)}


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("story", sorted(STORIES))
def test_moment_checkpoint(story, walls):
    from paper_1109_3277_amd.binding import Lattice

    dims = (34, 25, 27)
    ra, rb = W.layered_fields(dims, 91)
    groups = {"add0": (np.array([[5.0, 3.0], [4.0, 4.0]]), np.array([[9.3, 8.1, 13.4], [24.6, 16.2, 12.7]]),
                       np.array([[0.9, 0.2, 0.3, 0.1], [1.0, 0.0, 0.0, 0.0]]), np.array([0.2, -0.2]), np.array([2.0, 1.0])),
              "add1": (np.array([[3.0, 4.5]]), np.array([[16.4, 8.8, 14.1]]), np.array([[0.3, 0.9, 0.2, -0.1]]),
                       np.array([0.1]), np.array([1.5]))}
    log(f"case {story} walls={walls}")

    def handle():
        g = Lattice(dims, 1.0, 0.08, 1, "fp64", max_particles=3, max_radius=5.0)
        if walls:
            g.set_static_solid(W.wall_mask(dims), (0.01, -0.005, 0.0))
        return g

    a, force = handle(), None
    for act in STORIES[story]:
        if act == "init":
            a.init_fields(ra, rb, np.tile([0.01, -0.02, 0.005], (a.N, 1)))
        elif act == "save":
            a.save_state()
        elif act == "reload":
            a.load_state(a.save_state())
        elif act in groups:
            a.add_ellipsoids(*groups[act])
        elif act in FORCES:
            force = FORCES[act]
            a.set_body_accel(force)
        else:
            a.step(act)
    before = a.read_fields()
    image = a.save_state()
    assert all(np.array_equal(x, y) for x, y in zip(before, a.read_fields()))
    b = handle()
    b.load_state(image)
    if force is not None:
        b.set_body_accel(force)
    assert all(np.array_equal(x, y) for x, y in zip(before, b.read_fields()))
    assert _digest(b.save_state()) == _digest(image)
    for n in (1, 8):
        a.step(n)
        b.step(n)
        for x, y in zip(a.read_fields(), b.read_fields()):
            assert np.array_equal(x, y)
        pa, pb = a.read_particles(), b.read_particles()
        for k in pa:
            assert np.array_equal(pa[k], pb[k]), k
    assert _digest(a.save_state()) == _digest(b.save_state())
    a.close()
    b.close()


def test_thin_box_enqueues_without_planning():
    """A long thin box: the split of its planes over the blocks is not worked out
    again on the host in every step (it was, plane count by plane count: some
    4 ms a step here). Enqueueing a step takes a few microseconds; 1 ms allows
    for a slow host."""
    import time

    import torch
    from paper_1109_3277_amd.binding import Lattice

    dims = (3, 3, 1 << 20)
    g = Lattice(dims, 1.0, 0.08, 1, "fp64")
    ra = np.full(g.N, 0.7)
    g.init_fields(ra, ra)
    g.step(2)
    steps, best = 10, 1e9
    for _ in range(3):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        g.step_async(steps)
        best = min(best, (time.perf_counter() - t0) / steps)
    torch.cuda.synchronize()
    log(f"  {1e6 * best:.1f} us per step to enqueue")
    assert best < 1e-3
    g.close()
