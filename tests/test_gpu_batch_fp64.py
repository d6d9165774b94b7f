"""FP64 batches whose systems step in moments (tau = 1) and in populations
(tau != 1) side by side, without solids, with particles and with walls: steps,
tuning and checkpoints against lone handles, bit for bit."""
import hashlib

import numpy as np
import pytest

from paper_1109_3277_amd import workloads as W
from tests.parity_util import log

pytestmark = pytest.mark.gpu


def _specs(taus, dims0):
    """Four systems: ellipsoids, ellipsoids, no solids, walls; one tau each."""
    out = []
    for k, tau in enumerate(taus):
        dims = tuple(d + 2 * k for d in dims0)
        ra, rb = W.layered_fields(dims, 70 + k)
        parts = None
        if k < 2:
            parts = (np.array([[5.0, 3.0], [3.0, 4.0]]),
                     np.array([[8.3, 7.1, dims[2] / 2 - 0.4], [dims[0] - 7.6, dims[1] - 8.2, dims[2] / 2 + 1.1]]),
                     np.array([[0.9, 0.2, 0.3, 0.1], [0.4, -0.5, 0.6, 0.2]]), np.array([0.1, -0.1]), np.array([2.0, 4.0]))
        out.append(dict(dims=dims, tau=tau, ra=ra, rb=rb, parts=parts, walls=k == 3))
    return out


def _set(h, s):
    if s["walls"]:
        h.set_static_solid(W.wall_mask(s["dims"]), (0.01, 0.0, -0.004))
    h.init_fields(s["ra"], s["rb"])
    h.set_body_accel((1e-5, -2e-5, 0.0))
    if s["parts"]:
        h.add_ellipsoids(*s["parts"])


def _args(s):
    return {"dims": s["dims"], "tau": s["tau"], "g_br": 0.08, "psi_kind": 1,
            "max_particles": 2 if s["parts"] else 0, "max_radius": 5.0 if s["parts"] else 0.0}


def _batch(specs):
    from paper_1109_3277_amd.binding import Batch

    b = Batch([_args(s) for s in specs], "fp64")
    for k, s in enumerate(specs):
        _set(b[k], s)
    return b


def _lone(s):
    from paper_1109_3277_amd.binding import Lattice

    g = Lattice(precision="fp64", **_args(s))
    _set(g, s)
    return g


def _same(a, b, what):
    for k, (x, y) in enumerate(zip(a.read_fields(), b.read_fields())):
        assert np.array_equal(x, y), (what, "field", k)
    pa, pb = a.read_particles(), b.read_particles()
    for k in pa:
        assert np.array_equal(pa[k], pb[k]), (what, k)
    assert np.array_equal(a.stats(), b.stats()), (what, "stats")


def _image(g):
    return hashlib.sha256(g.save_state()).hexdigest()


def test_batch_of_both_paths_tuned_and_saved():
    specs = _specs((1.0, 1.25, 1.0, 1.25), (33, 25, 24))
    log(f"case mixed taus {[(s['dims'], s['tau']) for s in specs]}")
    b, lone = _batch(specs), [_lone(s) for s in specs]
    for k, g in enumerate(lone):
        _same(b[k], g, f"system {k}, no step")
        assert _image(b[k]) == _image(g), k
    done = 0
    for n in (3, 2, 4):  # an odd parity at the first tuning
        b.step(n)
        done += n
        for k, g in enumerate(lone):
            g.step(n)
            _same(b[k], g, f"system {k} after {done} steps")
            assert _image(b[k]) == _image(g), f"image of system {k} after {done} steps"
        if done == 3:
            assert not b.tune_report()["cached"]
            for k, g in enumerate(lone):
                _same(b[k], g, f"system {k} after tuning")
                assert _image(b[k]) == _image(g), f"image of system {k} after tuning"
    b.close()


def test_tuning_before_the_first_step_and_particles_after_it():
    """Tuned straight after the fields were set; particles placed over the tuned
    state, saved, and stepped."""
    specs = _specs((1.0, 1.25, 1.0, 1.25), (37, 23, 22))
    parts = [s["parts"] for s in specs]
    for s in specs:
        s["parts"] = None
    log(f"case tuned first {[(s['dims'], s['tau']) for s in specs]}")
    args = [dict(_args(s), max_particles=2 if p else 0, max_radius=5.0 if p else 0.0) for s, p in zip(specs, parts)]
    from paper_1109_3277_amd.binding import Batch, Lattice

    b, lone = Batch(args, "fp64"), [Lattice(precision="fp64", **a) for a in args]
    for k, s in enumerate(specs):
        _set(b[k], s)
        _set(lone[k], s)
    assert not b.tune_report()["cached"]
    for k, p in enumerate(parts):
        _same(b[k], lone[k], f"system {k} tuned")
        if p:
            b[k].add_ellipsoids(*p)
            lone[k].add_ellipsoids(*p)
        assert _image(b[k]) == _image(lone[k]), f"image of system {k}"
    b.step(5)
    for k, g in enumerate(lone):
        g.step(5)
        _same(b[k], g, f"system {k}")
        assert _image(b[k]) == _image(g), f"image of system {k} after steps"
    b.close()


def test_states_set_again_at_an_odd_step():
    """Fields, a checkpoint and a body force set on single systems of a batch whose
    copies stand at the odd parity."""
    specs = _specs((1.0, 1.25, 1.0, 1.25), (34, 22, 25))
    log(f"case set again {[(s['dims'], s['tau']) for s in specs]}")
    b, lone = _batch(specs), [_lone(s) for s in specs]
    early = [g.save_state() for g in lone]
    b.step(3)
    for k, g in enumerate(lone):
        g.step(3)
        for h in (b[k], g):
            if k in (0, 1):
                h.init_fields(specs[k]["rb"], specs[k]["ra"], np.tile([0.01, -0.02, 0.005], (h.N, 1)))
            else:
                h.load_state(early[k])
                h.set_body_accel((0.0, 3e-5, -1e-5))
        _same(b[k], g, f"system {k} set again")
        assert _image(b[k]) == _image(g), k
    for n in (2, 3):
        b.step(n)
        for k, g in enumerate(lone):
            g.step(n)
            _same(b[k], g, f"system {k}")
            assert _image(b[k]) == _image(g), k
    b.close()


def test_tune_cache_keeps_the_two_paths_apart():
    """Boxes and solids alike, one batch in moments and one in populations: each
    is timed for its own kernel, and only a batch of the same kind takes its
    choice."""
    seen = []
    for tau in (1.0, 1.25, 1.0, 1.25, 1.5):
        specs = _specs((tau,) * 4, (35, 21, 23))
        b = _batch(specs)
        seen.append(b.tune_report())
        log(f"  tau {tau}: {seen[-1]}")
        b.close()
    assert [r["cached"] for r in seen] == [False, False, True, True, True]
    assert seen[2]["candidates"] == seen[0]["candidates"] and seen[3]["candidates"] == seen[1]["candidates"]
