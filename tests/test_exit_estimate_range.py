"""When the FP64 kernels trust their FP32 exit-time estimates (CPU).

An estimate is bounded by 1.5e-6 only while its FP32 operands and results are normal numbers, so the kernel
takes it as sure only inside ranges that it tests with two comparisons: m, the smaller of the distance and the
logarithm's argument, and m |u_p| from below, and the estimate from below.  Every other bound follows from
these, and the divisions of the exit time evaluated afterwards rely on them.  The thresholds are read from
the kernel's source; the estimate is emulated in float32 with the hardware's reciprocal and logarithm moved
by up to the 2 ulp measured for them.
"""
import os
import re

import numpy as np
import pytest

from .test_fp32_estimates import BOUND, F, estimate

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "paper_2302_13590_amd", "csrc", "pt_kernels.hip")


def _thresholds():
    """(min of m and m |u_p|, E) of the kernel's rule; fails when the rule has another form."""
    src = open(SOURCE).read()
    m = re.search(r"const float m = fminf\(fabsf\(Df\), q\);\s+"
                  r"sure = \(int\)\(fminf\(m, m \* fabsf\(upf\)\) >= (\S+)f\) & \(int\)\(E >= (\S+)f\);", src)
    assert m, "exit_estimate no longer decides `sure` in the form that this test emulates"
    return tuple(float.fromhex(v) for v in m.groups())


LOW, LOW_E = _thresholds()


def _sure(D, up, A, ue, rng):
    """The estimate, the kernel's verdict on it, and whether it takes the ratio form."""
    with np.errstate(all="ignore"):
        E = estimate(D, up, A, ue, rng)
        Df, upf = D.astype(F), up.astype(F)
        rup = (F(1.0) / upf).astype(F)
        xf = (A.astype(F) * (Df * rup).astype(F)).astype(F)
        ratio = ~(xf > F(-0.5))
        q = np.where(ratio, (ue.astype(F) * rup).astype(F), (F(1.0) + xf).astype(F))
        # fminf passes a NaN by, comparisons with one fail
        m = np.fmin(np.abs(Df), q)
        sure = (np.fmin(m, (m * np.abs(upf)).astype(F)) >= F(LOW)) & (E >= F(LOW_E))
    return E, sure, ratio


def _exact(D, up, A, ue):
    with np.errstate(all="ignore"):
        x = A * (D / up)
        dt = np.where(x < -0.5, np.log(ue / up) / A, (D / up) * np.where(np.abs(x) < 1e-9, 1.0 - x / 2.0, np.log1p(x) / x))
    return x, dt


def _draw(rng, n):
    """Operands of feasible axes on both sides of every threshold: D, u_p, A, u_e."""
    sign = rng.choice([-1.0, 1.0], n)
    up = sign * 2.0 ** np.where(rng.random(n) < 0.5, rng.uniform(-130, 130, n), rng.uniform(-40, 40, n))
    near = np.log2(LOW) - np.minimum(np.log2(np.abs(up)), 0.0) + rng.uniform(-5, 5, n)   # m or m |u_p| at the threshold
    D = np.minimum(1.0, 2.0 ** np.choose(rng.integers(0, 3, n), [near, rng.uniform(-160, 0.5, n), rng.uniform(-20, 0.5, n)])) * sign
    # u_e / u_p: strong deceleration (around the threshold), uniform, acceleration up to where x overflows FP32
    ratio = 2.0 ** np.choose(rng.integers(0, 4, n), [np.minimum(near, 0.0), rng.uniform(-160, 0, n), rng.uniform(-3, 3, n),
                                                     rng.uniform(0, 200, n)])
    ratio = np.where(rng.random(n) < 0.1, 1.0 + 2.0 ** rng.uniform(-60, -20, n), ratio)
    with np.errstate(all="ignore"):
        ue = up * ratio
        A = (ue - up) / np.abs(D) * sign   # so that the particle reaches u_e after D
    ok = np.isfinite(ue) & np.isfinite(A) & (ue != 0) & (D != 0)
    return D[ok], up[ok], A[ok], ue[ok]


def test_trusted_estimates_and_what_follows_from_them():
    rng = np.random.default_rng(2024)
    trusted = total = 0
    assert LOW >= 2.0 ** -126                                   # D, q, u_p and u_e = q u_p: normal FP32 numbers
    top = 84.0 / LOW_E                                          # D / u_p >= E / 84, D <= 1
    worst = 0.0
    near = 0
    for _ in range(8):
        D, up, A, ue = _draw(rng, 250_000)
        E, sure, ratio = _sure(D, up, A, ue, rng)
        x, dt = _exact(D, up, A, ue)
        keep = sure & (dt > 0)
        assert np.array_equal(keep, sure)                       # nothing trusted without an exit
        Es = E[sure].astype(np.float64)
        assert np.isfinite(Es).all()
        worst = max(worst, float(np.abs(Es / dt[sure] - 1.0).max()))
        # what exit_time64_fast's divisions rely on
        assert 0.99 * LOW <= np.abs(up[sure]).min() and np.abs(up[sure]).max() <= top <= 2.0 ** 107
        assert 0.99 * LOW <= np.abs(D[sure]).min() and np.abs(D[sure]).max() <= 1.0
        assert np.abs(ue[sure & ratio]).min() >= 0.99 * LOW
        assert np.abs(x[sure]).max() < 2.0 ** 128
        trusted += int(sure.sum())
        total += sure.size
        near += int((np.log2(np.abs(D[sure]) * np.minimum(1.0, np.abs(up[sure])) / LOW) < 1).sum())
    assert worst < BOUND, worst
    assert total // 20 < trusted < total // 2 and near > 1000   # both verdicts, and next to the thresholds


@pytest.mark.parametrize("D, up, A, ue", [
    (0.0, 1.0, 0.5, 1.5),                 # on the face already
    (0.0, 1.0, 1e39, 2.0),                # and a gradient beyond FP32: inf * 0
    (0.0, 1e-50, 0.0, 1e-50),             # and a velocity that rounds to zero: 0 * inf
    (0.5, 1e-50, 1.0, 1.0), (0.5, 1e-41, 1.0, 1.0),      # u_p that rounds to zero, FP32-subnormal
    (0.5, 1e39, -1e39, 1e39), (0.5, 1e20, -4e39, -1e39),  # u_p, the gradient beyond FP32
    (1e-44, 1.0, 1.0, 2.0),               # distance FP32-subnormal
    (0.5, -1.0, 1e38, -1e-45),            # ratio form, u_e below FP32
    (0.5, 1.0, np.inf, np.inf), (0.5, np.inf, np.inf, np.inf), (0.5, np.inf, np.nan, np.inf),
    (0.5, np.nan, 1.0, 1.0), (np.nan, 1.0, 1.0, 1.0), (0.5, 1.0, np.nan, 1.0),
    (1.0, LOW / 2, 0.0, LOW / 2),         # just below each threshold
    (LOW / 2, 1.0, 0.0, 1.0),
    (1.0, 1.0, LOW / 2 - 1.0, LOW / 2),
    (1.0, 2 / LOW_E, 0.0, 2 / LOW_E),
], ids=str)
def test_never_trusted(D, up, A, ue):
    rng = np.random.default_rng(5)
    E, sure, _ = _sure(*(np.array([v], dtype=np.float64) for v in (D, up, A, ue)), rng)
    assert not sure[0], E


@pytest.mark.parametrize("D, up, A, ue", [
    (1.0, 2 * LOW, 0.0, 2 * LOW), (2 * LOW_E, 1.0, 0.0, 1.0), (1.0, 1.0, -1.0, 2 * LOW),
    (1.0, 0.5 / LOW_E, 0.0, 0.5 / LOW_E), (-0.5, -1.0, 0.0, -1.0)], ids=str)
def test_trusted_just_inside(D, up, A, ue):
    rng = np.random.default_rng(6)
    E, sure, _ = _sure(*(np.array([v], dtype=np.float64) for v in (D, up, A, ue)), rng)
    assert sure[0], E


@pytest.mark.parametrize("jump, scale", [(1.0, 1e-27), (1e-6, 1e-24), (1e-12, 1e-20), (1e-12, 1e-9), (1e-12, 1.0),
                                         (1e-12, 1e14), (1e-12, 1e22)])
def test_trusted_in_any_unit_of_time(jump, scale):
    """Ordinary steps, also towards a face that is 1e12 times slower, are trusted whatever unit the
    velocities are in: nothing but the margin sends them to three exact exit times."""
    rng = np.random.default_rng(7)
    n = 20_000
    up = scale * rng.uniform(0.01, 10.0, n)
    D = rng.uniform(1e-6, 1.0, n)
    ue = up * jump * rng.uniform(0.5, 1.0, n)
    E, sure, _ = _sure(D, up, (ue - up) / D, ue, rng)
    assert sure.all()
