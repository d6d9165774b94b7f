"""lb_step's verdict on a run that goes bad: a density that turns negative during
a step from sound fields (strong interaction), in a lone system without solids,
with walls and with a particle, and in one system of a batch; and bad densities
that were set, loaded, set over, or covered by solids before the first step."""
import numpy as np
import pytest

from paper_1109_3277_amd import workloads as W
from tests.parity_util import log

pytestmark = pytest.mark.gpu

DIMS = (24, 20, 18)
PARTICLE = (np.array([[5.0, 3.0]]), np.array([[12.2, 10.3, 9.1]]), np.array([[0.9, 0.2, 0.3, 0.1]]), np.array([0.0]),
            np.array([1e6]))


def _fields():
    return W.uniform_fields(DIMS, 5, 0.7, 0.7, 0.05)


def _args(kind, tau=1.0, g_br=0.08):
    return {"dims": DIMS, "tau": tau, "g_br": g_br, "psi_kind": 1, "max_particles": 1 if kind == "particle" else 0,
            "max_radius": 5.0 if kind == "particle" else 0.0}


def _set(h, kind, ra, rb):
    if kind == "walls":
        h.set_static_solid(W.wall_mask(DIMS))
    h.init_fields(ra, rb)
    if kind == "particle":
        h.add_ellipsoids(*PARTICLE)


def _bad(h):
    ra, rb, _, own = h.read_fields()
    fl = own == -1
    return not (ra[fl].min() >= 0.0 and rb[fl].min() >= 0.0)


def _refused(step):
    """The message of the LB_EUNSTABLE that `step()` raises, None if it returns."""
    from paper_1109_3277_amd.binding import LB_EUNSTABLE, LBError

    try:
        step()
    except LBError as e:
        assert e.code == LB_EUNSTABLE
        return str(e)
    return None


@pytest.mark.parametrize("prec,tau", [("fp64", 1.0), ("fp64", 1.25), ("fp32", 1.0)])
@pytest.mark.parametrize("kind", ["plain", "walls", "particle"])
def test_density_gone_bad_during_a_step(kind, prec, tau):
    from paper_1109_3277_amd.binding import Lattice

    log(f"case gone bad {kind} {prec} tau={tau}")
    g = Lattice(precision=prec, **_args(kind, tau, 0.3))
    _set(g, kind, *_fields())
    first = None
    for k in range(1, 41):
        msg = _refused(lambda: g.step(1))
        if first is None and _bad(g):
            first = k
        if msg:
            break
        # populations are looked at when the next step begins where there are no
        # particles; moments as they are formed
        moments = prec == "fp64" and tau == 1.0
        assert first is None or (not moments and k == first), k
    log(f"  bad at step {first}, reported at {k}: {msg}")
    assert msg and "negative density" in msg and first is not None and k - first <= 1
    assert g.stats()[7] == 1.0
    assert _refused(lambda: g.step(0))  # it stays reported
    g.close()


def test_one_system_of_a_batch_gone_bad():
    from paper_1109_3277_amd.binding import Batch

    specs = [("particle", 1.0, 0.08), ("particle", 1.0, 0.3), ("plain", 1.0, 0.08), ("walls", 1.25, 0.08)]
    log(f"case batch gone bad {specs}")
    b = Batch([_args(*s) for s in specs], "fp64")
    for k, s in enumerate(specs):
        _set(b[k], s[0], *_fields())
    for n in range(1, 41):
        msg = _refused(lambda: b.step(1))
        assert bool(msg) == _bad(b[1]), n
        if msg:
            break
    log(f"  step {n}: {msg}")
    assert msg and "system 1" in msg
    assert [b[k].stats()[7] for k in range(4)] == [0.0, 1.0, 0.0, 0.0]
    b.close()


@pytest.mark.parametrize("prec,tau", [("fp64", 1.0), ("fp64", 1.25), ("fp32", 1.0)])
@pytest.mark.parametrize("kind", ["plain", "walls", "particle"])
def test_bad_density_that_was_set(kind, prec, tau):
    """Reported by the first step, lone and batched; not if other fields are set
    before it."""
    from paper_1109_3277_amd.binding import Batch, Lattice

    ra, rb = _fields()
    worse = ra.copy()
    worse.reshape(DIMS[::-1])[3, 2, 1] = -0.01  # fluid in every kind
    log(f"case set bad {kind} {prec} tau={tau}")
    g = Lattice(precision=prec, **_args(kind, tau))
    b = Batch([_args("plain", tau), _args(kind, tau)], prec)
    b[0].init_fields(ra, rb)
    for h in (g, b[1]):
        _set(h, kind, worse, rb)
    assert g.stats()[7] == 1.0 and _refused(lambda: g.step(0)) is None
    image = g.save_state()
    assert _refused(lambda: g.step(1))
    assert "system 1" in _refused(lambda: b.step(1))
    # an image of the bad state, then one of a good state, in a handle of its own
    a = Lattice(precision=prec, **_args(kind, tau))
    a.load_state(image)
    assert _refused(lambda: a.step(1))
    g = Lattice(precision=prec, **_args(kind, tau))
    _set(g, kind, ra, rb)
    a.load_state(g.save_state())
    assert _refused(lambda: a.step(2)) is None
    # set over before any step
    g = Lattice(precision=prec, **_args(kind, tau))
    _set(g, kind, worse, rb)
    g.init_fields(ra, rb)
    assert _refused(lambda: g.step(2)) is None
    b.close()


@pytest.mark.parametrize("prec,tau", [("fp64", 1.0), ("fp64", 1.25)])
@pytest.mark.parametrize("value", [-0.5, float("nan")])
def test_bad_density_under_a_particle_is_of_no_account(value, prec, tau):
    """Fields without meaning where a particle is then placed: lone, batched, and
    through a checkpoint."""
    from paper_1109_3277_amd.binding import Batch, Lattice

    ra, rb = _fields()
    worse = ra.copy()
    worse.reshape(DIMS[::-1])[8:11, 9:12, 11:14] = value
    log(f"case covered {value} {prec} tau={tau}")
    out = []
    for loaded in (False, True):
        g = Lattice(precision=prec, **_args("particle", tau))
        g.init_fields(worse, rb)
        if loaded:
            image = g.save_state()
            g = Lattice(precision=prec, **_args("particle", tau))
            g.load_state(image)
        g.add_ellipsoids(*PARTICLE)
        assert not _bad(g)
        assert _refused(lambda: g.step(5)) is None
        out.append(g.read_fields())
    b = Batch([_args("particle", tau)], prec)
    _set(b[0], "particle", worse, rb)
    assert _refused(lambda: b.step(5)) is None
    out.append(b[0].read_fields())
    for f in out[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(out[0], f))
    good = Lattice(precision=prec, **_args("particle", tau))
    _set(good, "particle", ra, rb)
    good.step(5)
    assert all(np.array_equal(x, y) for x, y in zip(out[0], good.read_fields()))
    b.close()
