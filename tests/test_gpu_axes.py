"""FP64 parity of the one-lane-per-axis kernel (the library's own launch for few particles) with the
oracle: the sizes at which its quads, waves and blocks are ragged and at which it gives way to one
lane per particle, every output mode, limits, directions, groups and transient flow, and the
per-cell edge cases of the other kernels.  Results must be bitwise the oracle's, as theirs are.
"""
import math

import numpy as np
import pytest

from oracle import oracle as O
from workloads import configs as C

from . import test_gpu_edge_cases as E
from . import test_gpu_pathline as L
from . import test_gpu_transient as T
from .gpu_util import compare, gpu_track, require_gpu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
SP = (10.0, 10.0, 2.0)


@pytest.fixture(scope="module")
def pt():
    return require_gpu()


def _grid():
    return L.CASES["lognormal_wells"]()


def _release(n, g, seed):
    return C.release(np.random.Generator(np.random.PCG64(seed)), n, g.nx, g.ny, g.nz)


@pytest.mark.parametrize("n", [0, 1, 15, 16, 17, 63, 64, 65, 1001])
@pytest.mark.parametrize("direction", [1, -1])
def test_ragged_sizes(pt, n, direction):
    g = _grid()
    p = _release(n, g, 7 + n)
    r = O.track(g, p, direction=direction)
    for kw in (dict(), dict(use_graph=1), dict(sort=2)):
        out = gpu_track([g], p, direction=direction, **kw)
        compare(out, r, label="n %d %s" % (n, kw), spacing=SP)
        assert out["summary"]["crossings"] == int(r.ncross.sum())


def test_hand_over_to_one_lane_per_particle(pt):
    """At 128 particles per compute unit the launch still takes four lanes each, one more does not;
    both give the same results."""
    g = _grid()
    n = 128 * torch.cuda.get_device_properties(0).multi_processor_count
    p = _release(n + 1, g, 3)
    few = gpu_track([g], p.subset(np.arange(n)))
    many = gpu_track([g], p)
    assert few["summary"]["grid"] * few["summary"]["block"] == 4 * n
    assert many["summary"]["grid"] * many["summary"]["block"] < 4 * n
    for k in ("cell", "xi", "eta", "zeta", "t", "status", "ncross", "path_hash", "out_xyz"):
        assert np.array_equal(few[k], many[k][:n], equal_nan=True), k
    idx = np.arange(0, n, 41)
    compare(few, O.track(g, p.subset(idx)), idx=idx, label="hand-over", spacing=SP)


@pytest.mark.parametrize("t_max", [math.inf, 700.0])
def test_timeseries(pt, t_max):
    g = _grid()
    p = _release(1003, g, 17)
    p.t[:] = np.random.Generator(np.random.PCG64(18)).choice([0.0, 3.0, 50.0], size=p.n)
    snaps = np.concatenate([[0.0, 0.5], np.logspace(0, 3.5, 37), [5000.0, 5000.0]])
    r = O.track(g, p, snap_times=snaps, t_max=t_max)
    compare(gpu_track([g], p, snap_times=snaps, t_max=t_max), r, label="ts", spacing=SP)


@pytest.mark.parametrize("kw", [dict(), dict(direction=-1), dict(t_max=400.0), dict(max_steps=9), dict(stop_at_sink=0)],
                         ids=str)
def test_pathlines(pt, kw):
    g = _grid()
    p = _release(517, g, 23)
    r, offs, flat = L.oracle_paths(g, p, **kw)
    out, paths = L.gpu_pathlines(pt, [g], p, **kw)
    compare(out, r, label="pathlines %s" % kw, spacing=SP)
    L.compare_paths(paths, offs, flat, "pathlines %s" % kw)


def test_groups_and_transient(pt):
    grids = [C.random_grid(12, 9, 4, s2, 2.0, 300 + q, recharge=1e-3 * q) for q, s2 in enumerate((0.5, 1.5, 3.0))]
    offs, gg = np.array([0, 70, 70, 71, 195]), np.array([2, 0, 1, 0], np.int32)
    p = C.concat([_release(int(m), grids[q], 60 + q) for m, q in zip(np.diff(offs), gg)])
    snaps = np.logspace(-1, 3, 20)
    for kw in (dict(), dict(snap_times=snaps, t_max=300.0)):
        r = O.track_groups(grids, p, offs, gg, **kw)
        compare(gpu_track(grids, p, group_offsets=offs, group_grid=gg, **kw), r, label="groups %s" % kw, spacing=SP)
    fields = T._fields()
    p = T._staged(1001, fields[0], 11)
    for kw in (dict(stop_at_sink=1), dict(stop_at_sink=0, t_max=120.0), dict(snap_times=np.linspace(0.0, 900.0, 41), t_max=900.0)):
        r = O.track_transient(fields, T.ENDS, p, **kw)
        compare(gpu_track(fields, p, tstep_end=T.ENDS, **kw), r, label="transient %s" % kw, spacing=SP)


@pytest.mark.parametrize("case", sorted(k for k in vars(E) if k.startswith("test_")))
def test_edge_cases_of_the_other_kernels(pt, case, monkeypatch):
    """Every edge-case test of the other kernels, run through the library's own launch."""
    own = [dict(), dict(use_graph=1)]
    monkeypatch.setattr(E, "FORMS", own)
    monkeypatch.setattr(E._parity, "__defaults__", (own,) + E._parity.__defaults__[1:])
    test = getattr(E, case)
    marks = [m for m in getattr(test, "pytestmark", []) if m.name == "parametrize"]
    for value in (marks[0].args[1] if marks else [None]):
        test(pt, value) if marks else test(pt)
