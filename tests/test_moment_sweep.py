"""The box sweep's form of the single-precision moments (CPU only).

moments_single<true> in paper_2102_01734_amd/csrc/fs_point.hpp returns h = D e1 - e2
in place of e2.  Its operations, replayed in double precision with correctly
rounded FMAs, stay as close to 40-digit values as the e2 form is required to
(1e-12 for ex and e0, 1e-10 for e1 and h), on both sides of the n = 0 choice, and
half depths added with kMinStep / 2 each give the optical step bit for bit."""
import math

import mpmath
import numpy as np
import pytest

from tests.test_moment_poly import _fma, _gen

mpmath.mp.dps = 40


def _moments(D, c):
    z = min(D, 745.0)
    n = float(np.rint(z * 1.4426950408889634))
    r = _fma(n, -0.6931471805599453, z)
    P = _fma(c[6], -r, c[5])
    for k in (4, 3, 2, 1, 0):
        P = _fma(P, -r, c[k])
    r2 = r * r
    q = _fma(-r, P, 0.5)
    if n == 0.0:
        e1 = r2 * q
        e0 = D - e1
        return 1.0 - e0, e0, e1, (D * r2) * _fma(-2.0, P, q)
    ex = math.ldexp(_fma(r2, q, 1.0 - r), -int(n))
    e0 = 1.0 - ex
    e1 = D - e0
    return ex, e0, e1, _fma(2.0, e1, -(D * e0))


@pytest.mark.parametrize("D", sorted([1e-12, 1e-9, 1e-5, 0.02, 0.3, 0.3465, 0.34657, 0.34658, 0.4, 1.0, 1.039, 1.04,
                                      2.0, 10.0, 104.0, 700.0, 744.0, 1e4, 1e20]))
def test_sweep_moments_accuracy(D):
    Dm = mpmath.mpf(D)
    e0 = -mpmath.expm1(-Dm)
    e1 = Dm - e0
    ref = (mpmath.exp(-Dm), e0, e1, 2 * e1 - Dm * e0)
    got = _moments(D, [float(v) for v in _gen().coefficients()])
    for name, g, r, tol in zip(("ex", "e0", "e1", "h"), got, ref, (1e-12, 1e-12, 1e-10, 1e-10)):
        assert abs(g - float(r)) <= tol * abs(float(r)) + 1e-300, (name, D, g, float(r))


def test_half_depths_sum_to_the_optical_step():
    rng = np.random.default_rng(5)
    chi = (10.0 ** rng.uniform(-12, 12, (2, 4000))).astype(np.float32).astype(np.float64)
    s = rng.uniform(1e-3, 40.0, (2, 4000))
    half = [_fma_array(chi[k], 0.5 * s[k], 0.5e-100) for k in range(2)]
    assert np.array_equal(half[0] + half[1], 0.5 * (chi[0] * s[0] + chi[1] * s[1]))
    assert _fma(0.0, 1.0, 0.5e-100) * 2 == 1e-100


def _fma_array(a, b, c):
    return np.array([_fma(x, y, c) for x, y in zip(a, b)])
