"""The mixed-precision step's choice of the exit face, against the FP64 oracle.

Its three exit times are compared in FP32; an axis whose gradient is nearly zero enters with
D/u_p and is evaluated in double when it is the earliest or the choice is close.  The cases put
ties, near-zero gradients on both sides of the series' range, zero distances and unreachable faces
on every axis.  Face velocities and coordinates are FP32 numbers, so ties are ties in both
precisions and the cell, face (local coordinate on it), count and status have to be the oracle's.

Tolerance 2^-18: an exit time is a product of at most six FP32 roundings and three hardware
functions of 2 ulp (2^-20 in all); a coordinate moves by at most one cell by such a time and three
more functions.
"""
import itertools

import numpy as np
import pytest

from oracle import oracle as O

from . import helpers as H
from .gpu_util import gpu_track, require_gpu

pytestmark = pytest.mark.gpu

# (low face velocity, high face velocity, local coordinate) per axis
ONE = (1.0, 1.0, 0.5)
CASES = {
    "tie of three": (ONE, ONE, ONE),
    "tie, curved": ((1.0, 2.0, 0.25), (1.0, 2.0, 0.25), (0.25, 0.25, 0.5)),
    "tie, both directions": ((-2.0, -1.0, 0.75), (1.0, 2.0, 0.25), (0.0, 0.0, 0.5)),
    "near zero, close": ((1.0, 1.0 + 2.0 ** -12, 0.5), (1.0, 1.0 - 2.0 ** -12, 0.5), (1.0, 1.0 + 2.0 ** -14, 0.5)),
    "near zero and curved, close": ((1.0, 1.0 + 2.0 ** -8, 0.5), (1.0, 1.0 + 2.0 ** -10, 0.5), (1.0, 0.996, 0.5)),
    "near zero, far": ((1.0, 1.0 + 2.0 ** -13, 0.5), (0.25, 1.0, 0.5), (-0.125, -0.125, 0.5)),
    "near zero, later": ((0.125, 0.125, 0.5), (1.0, 3.0, 0.5), (0.0, 0.0, 0.25)),
    "edge of the series": ((1.0, 1.0 + 2.0 ** -9, 0.5), (0.5, 0.5 - 2.0 ** -10, 0.5), (0.25, 0.25, 0.5)),
    "on the exit face": ((1.0, 1.5, 1.0), (1.0, 1.0, 0.5), (0.5, 0.5, 0.5)),
    "on two exit faces": ((1.0, 1.0, 1.0), (-1.0, -1.0, 0.0), (0.5, 0.5, 0.5)),
    "strong deceleration": ((4.0, 2.0 ** -6, 0.0), (0.03125, 0.03125, 0.5), (0.0, 0.0, 0.5)),
    "stagnation": ((-1.0, 1.0, 0.5), (0.5, 0.5, 0.5), (1.0, -1.0, 0.25)),
    "no face": ((1.0, -1.0, 0.25), (0.0, 0.0, 0.5), (-1.0, 1.0, 0.5)),
    "small velocities": ((2.0 ** -110, 2.0 ** -110, 0.5), (2.0 ** -111, 2.0 ** -110, 0.5), (0.0, 0.0, 0.5)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_exit_choice(name):
    require_gpu()
    grids, parts = [], []
    for q in itertools.permutations(CASES[name]):
        g = H.box_grid(1, 1, 1, 1.0, 1.0, 1.0, porosity=1.0)
        (g.qx[0, 0, 0], g.qx[0, 0, 1], x), (g.qy[0, 0, 0], g.qy[0, 1, 0], y), (g.qz[0, 0, 0], g.qz[1, 0, 0], z) = q
        grids.append(g)
        parts.append((x, y, z))
    p = H.particles([0] * len(parts), *np.array(parts).T)
    offs, gg = np.arange(len(grids) + 1), np.arange(len(grids), dtype=np.int32)
    r = O.track_groups(grids, p, offs, gg)
    runs = [gpu_track(grids, p, group_offsets=offs, group_grid=gg, precision=1, schedule=s) for s in (1, 2)]
    one = [gpu_track([g], p.subset(np.arange(i, i + 1)), precision=1) for i, g in enumerate(grids)]
    runs.append({k: np.concatenate([o[k] for o in one]) for k in one[0] if k not in ("summary", "snap_xyz")})
    tol = 2.0 ** -18
    for out in runs:
        for k in ("cell", "status", "ncross", "path_hash"):
            assert np.array_equal(out[k], getattr(r, k)), (name, k)
        assert np.all(np.abs(out["t"] - r.t) <= tol * np.abs(r.t)), (name, out["t"], r.t)
        for k in ("xi", "eta", "zeta"):
            want = getattr(r, k)
            face = (want == 0.0) | (want == 1.0)
            assert np.array_equal(out[k][face], want[face]), (name, k, out[k], want)
            assert np.all(np.abs(out[k] - want) <= tol), (name, k, out[k], want)
