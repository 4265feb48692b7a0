"""Infinite face velocities, negative zeros and undecided roundings that a track does not need.

A flow field is checked for finite flows, but flow over pore volume can still overflow: the velocity of
a face is then infinite, and the method's formulas give NaN (inf - inf, inf * 0).  What the formulas give
is the result: a NaN coordinate stays NaN, and an exit time that is NaN is never the earliest.  The
oracle evaluates the formulas as they are written, so every kernel form must agree with it, NaN for NaN.
The same holds for the sign of a zero coordinate, and for what counts as a recheck: an evaluation whose
value the track does not use hands no particle to the careful pass.
"""
import itertools

import numpy as np
import pytest

from oracle import oracle as O

from . import helpers as H
from . import test_gpu_pathline as L
from .gpu_util import compare, gpu_track, require_gpu

pytestmark = pytest.mark.gpu

# one lane per axis (the library's own launch), static, persistent, face arrays, a captured launch
FORMS = [dict(), dict(schedule=1, layout=2), dict(schedule=2, layout=2), dict(schedule=1, layout=1), dict(use_graph=1)]
SNAPS = np.array([0.0, 0.3, 0.75, 1.0, 2.5, 7.0])
VOL = 1e-300     # dx dy dz of the cells below: a flow of 1e-300 is a velocity of 1, one above 2e8 is infinite


@pytest.fixture(scope="module")
def pt():
    return require_gpu()


def _grid(nx, ny, nz):
    return H.box_grid(nx, ny, nz, 1e-100, 1e-100, 1e-100, porosity=1.0)


def _same_sign(a, b):
    return np.array_equal(np.signbit(a) | np.isnan(a), np.signbit(b) | np.isnan(b))


def _check(g, p, label, **kw):
    r = O.track(g, p, **kw)
    rs = O.track(g, p, snap_times=SNAPS, **kw)
    for f in FORMS:
        out = gpu_track([g], p, **f, **kw)
        compare(out, r, label="%s %s" % (label, f))
        assert out["summary"]["crossings"] == int(r.ncross.sum()), label
        for k in ("xi", "eta", "zeta"):
            assert _same_sign(out[k], getattr(r, k)), (label, f, k)
        compare(gpu_track([g], p, snap_times=SNAPS, **f, **kw), rs, label="%s %s, snapshots" % (label, f))
    return r


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("t_max", [np.inf, 2.25])
def test_nan_coordinates_stay_nan(pt, axis, t_max):
    """The first of three cells along an axis has infinite velocities of one sign on another one: the
    particle's coordinate there is NaN from the first step on, also in the cells after it, whose velocities
    are finite."""
    shape = [1, 1, 1]
    shape[axis] = 3
    g = _grid(*shape)
    q = [g.qx, g.qy, g.qz]
    other = (axis + 1) % 3
    q[axis][:] = VOL
    q[other][:] = 0.01 * VOL
    first = [slice(None)] * 3
    first[2 - axis] = 0
    q[other][tuple(first)] = 1e10
    loc = [[0.25, 0.5, 0.0], [0.5, 0.5, 1.0], [0.125, 0.0, 0.5], [1.0, 0.75, 0.25]]
    xs = [np.roll(v, axis) for v in loc]
    p = H.particles([0] * len(xs), *np.array(xs).T)
    r = _check(g, p, "axis %d" % axis, t_max=t_max, max_steps=50)
    assert np.isnan(getattr(r, ("xi", "eta", "zeta")[other])).all()
    assert r.ncross.min() == (3 if np.isinf(t_max) else 2)


@pytest.mark.parametrize("t_max", [np.inf, 1.5])
def test_no_face_is_reached_in_nan_time(pt, t_max):
    """Velocities that grow to infinity along every axis: each exit time is NaN, so no face is reachable
    and the particle strands -- at the time limit when there is one -- without a crossing."""
    g = _grid(2, 2, 2)
    for q, a in ((g.qx, 2), (g.qy, 1), (g.qz, 0)):
        q[:] = VOL
        hi = [slice(None)] * 3
        hi[a] = slice(1, None)
        q[tuple(hi)] = 1e10
    p = H.particles([0, 0, 0], [0.5, 0.25, 0.75], [0.5, 0.125, 0.5], [0.5, 1.0, 0.25])
    r = _check(g, p, "nan exits", t_max=t_max, max_steps=50)
    assert (r.ncross == 0).all() and (r.status == 5).all()


def test_negative_zero_coordinates(pt):
    """A coordinate of -0.0 on an axis without motion keeps its sign, one that moves becomes what the sum
    gives; on the exit axis it is the face."""
    g = H.box_grid(4, 2, 2, 1.0, 1.0, 1.0, porosity=1.0)
    g.qx[:] = 1.0
    g.qy[:, :, 2:] = 1e-3
    nz = -0.0
    p = H.particles([0, 0, 0, 1, 0], [nz, 0.5, 0.25, nz, nz], [nz, nz, 0.5, nz, 0.0], [nz, 0.0, nz, 0.5, nz])
    for kw in (dict(), dict(t_max=0.5), dict(t_max=1.25), dict(direction=-1, t_max=3.0), dict(max_steps=1)):
        r = _check(g, p, "negative zero %s" % kw, **kw)
    assert np.signbit(r.zeta[0])
    g.qx[:] = 0.0
    g.qy[:] = 0.0
    _check(g, p, "negative zero, no flow", t_max=1.0)


def test_sign_of_a_zero_exit_time(pt):
    """Axes that leave at once, in a tie: a face at 0 is reached in -0.0, one at 1 in +0.0.  The step takes the
    time of the axis it leaves through, the lowest, and its sign decides that of a -0.0 on the other axes."""
    g = H.box_grid(3, 3, 3, 1.0, 1.0, 1.0, porosity=1.0)
    loc = np.array(list(itertools.product((0.0, -0.0, 0.5, 1.0), repeat=3)))
    for signs in itertools.product((1.0, -1.0), repeat=3):
        for q, s, a in zip((g.qx, g.qy, g.qz), signs, (0, 0, 0.125)):
            q[:] = s
            q[:, :, 1:] += a * s
        for t in (0.0, -0.0):
            p = H.particles([13] * len(loc), *loc.T)
            p.t[:] = t
            for steps in (1, 50):
                r = O.track(g, p, max_steps=steps)
                for f in FORMS:
                    out = gpu_track([g], p, max_steps=steps, **f)
                    compare(out, r, label="%s %s %s" % (signs, t, f))
                    for k in ("xi", "eta", "zeta", "t"):
                        assert _same_sign(out[k], getattr(r, k)), (signs, t, steps, f, k)


def _unit(q):
    """One cell of unit pore volume: face flows are velocities."""
    g = H.box_grid(1, 1, 1, 1.0, 1.0, 1.0, porosity=1.0)
    for a, (lo, hi) in zip((g.qx, g.qy, g.qz), q):
        a.reshape(-1)[:] = lo, hi
    return g


# velocities whose exp or log argument lies within 2^-96 of a rounding boundary (found by search)
UNDECIDED_EXIT = float.fromhex("0x1.0000000000006p+0")   # log1p(u2 - 1)
# expm1((u2 - u1) dt), dt the exit time from 0.75
UNDECIDED_ADVANCE = (float.fromhex("0x1.8000000000002p+1"), float.fromhex("0x1.7ffffffffffffp+1"))
UNUSED = {
    # no motion on x (u_p = 0), whose expm1(2^-52 * 1) is undecided; the limit comes first
    "axis at rest": (_unit([(-2.0 ** -53, 2.0 ** -53), (0.25, 0.25), (0.0, 0.0)]), (0.5, 0.25, 0.5), dict(t_max=1.0)),
    # leaves through x, where its coordinate is the face's whatever the advance to it would give
    "exit axis": (_unit([UNDECIDED_ADVANCE, (0.0, 0.0), (0.0, 0.0)]), (0.75, 0.5, 0.5), dict()),
    "exit axis, beside others": (_unit([(0.1, 0.1), UNDECIDED_ADVANCE, (0.1, 0.1)]), (0.0, 0.75, 0.5), dict()),
    # leaves through x four times sooner than through y, whose exit time is undecided
    "far axis": (_unit([(4.0, 4.0), (1.0, UNDECIDED_EXIT), (0.0, 0.0)]), (0.0, 0.0, 0.5), dict()),
}


@pytest.mark.parametrize("case", sorted(UNUSED))
def test_unused_evaluations_hand_nothing_over(pt, case):
    g, loc, kw = UNUSED[case]
    p = H.particles([0] * 3, *[[v] * 3 for v in loc])
    r = O.track(g, p, **kw)
    for f in FORMS:
        out = gpu_track([g], p, **f, **kw)
        compare(out, r, label="%s %s" % (case, f))
        assert out["summary"]["recheck_tracks"] == 0, (case, f, out["summary"]["recheck_tracks"])


@pytest.mark.parametrize("q, loc, kw", [
    ([(1.0, UNDECIDED_EXIT), (0.0, 0.0), (0.0, 0.0)], (0.0, 0.5, 0.5), dict()),                        # the exit time taken
    ([(1.0, UNDECIDED_EXIT), (1.0, UNDECIDED_EXIT), (0.0, 0.0)], (0.0, 0.0, 0.5), dict()),             # a tie
    ([(0.5, 0.5 + 2.0 ** -52), (0.25, 0.25), (0.0, 0.0)], (0.0, 0.25, 0.5), dict(t_max=1.0)),         # an advance to the limit
    ([(0.5, 0.5 + 2.0 ** -52), (1.0, 1.0), (0.0, 0.0)], (0.0, 0.0, 0.5), dict()),                      # another axis' advance
], ids=["exit time", "tie", "limit", "advance"])
def test_used_evaluations_are_handed_over(pt, q, loc, kw):
    """The other side: an undecided value that the track uses reaches the careful pass in every form."""
    g = _unit(q)
    p = H.particles([0] * 3, *[[v] * 3 for v in loc])
    r = O.track(g, p, **kw)
    for f in FORMS:
        out = gpu_track([g], p, **f, **kw)
        compare(out, r, label=str(f))
        assert out["summary"]["recheck_tracks"] == 3, f


def test_pathline_records_keep_nan(pt):
    g = _grid(3, 1, 1)
    g.qx[:] = VOL
    g.qy[:] = 0.01 * VOL
    g.qy[:, :, 0] = 1e10
    p = H.particles([0, 0], [0.25, 0.5], [0.5, 0.5], [0.5, 0.0])
    _, offs, flat = L.oracle_paths(g, p)
    for f in FORMS[:3]:
        _, paths = L.gpu_pathlines(pt, [g], p, **f)
        assert np.array_equal(paths["offsets"], offs)
        for k in ("t", "xyz", "cell", "face"):
            assert np.array_equal(paths[k], flat[k], equal_nan=paths[k].dtype.kind == "f"), (f, k)
