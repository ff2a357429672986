"""The entry of a span's best sample on the host (libbysdf_audit runs the
traversal's own functions): the scan that ranks the samples and the entry that
decides the hit form the ball's half chord in differently fused products, and
have to agree on whether the ball is met."""
import ctypes as C

import numpy as np
import pytest

import precision_audit as A
from paper_2401_12724_amd import build as hip_build


@pytest.fixture(scope="module", autouse=True)
def audit_lib():
    if hip_build.stale():
        hip_build.build()


def _spans(ctrl, o, d, nsamp):
    n = o.shape[1]
    sampled, entry = np.zeros(n), np.zeros(n)
    f = A.lib().bysdf_audit_span
    f.argtypes = [C.c_int64] + [C.c_void_p] * 3 + [C.c_int] + [C.c_void_p] * 2
    ctrl, o, d = (np.ascontiguousarray(x, np.float32) for x in (ctrl, o, d))
    assert f(n, A._ptr(ctrl), A._ptr(o), A._ptr(d), nsamp, A._ptr(sampled), A._ptr(entry)) == 0
    return sampled, entry


def test_tangent_rays():
    """Rays that touch a straight tube where a sample's ball is, in frames of
    integer vectors of integer length, so that all inputs are exact: the half
    chord squared is rounding noise of either sign, at most 32 ulps of R^2, so
    its root is below 1e-7 R."""
    a, b, c, e = np.random.default_rng(3).integers(-9, 10, (4, 20000))
    norm = a * a + b * b + c * c + e * e
    a, b, c, e, norm = (x[norm > 0] for x in (a, b, c, e, norm))
    d = np.stack([a * a + b * b - c * c - e * e, 2 * (b * c + a * e), 2 * (b * e - a * c)])
    p = np.stack([2 * (b * c - a * e), a * a - b * b + c * c - e * e, 2 * (c * e + a * b)])
    q = np.stack([2 * (b * e + a * c), 2 * (c * e - a * b), a * a - b * b - c * c + e * e])
    scale, n = 2.0 ** -10, len(norm)
    ctrl = np.zeros((4, n, 4))
    ctrl[:, :, :3] = np.arange(-1.5, 2.0)[:, None, None] * q.T * scale
    ctrl[:, :, 3] = norm * scale
    sampled, entry = _spans(ctrl, (p - 4 * d) * scale, d, 16)
    met = np.isfinite(sampled)
    assert met.sum() > 1000
    assert not np.isnan(entry).any()
    assert np.all(np.abs(entry[met] - sampled[met]) <= 1e-7 * (norm * scale)[met])


def test_sample_root():
    """The root in a sample's entry, refined from an estimate of 24 bits, is
    within an ulp of the rounded root over the half chords squared of tubes
    from 1e-6 to 1e3 in radius, down to touching rays."""
    x = 10.0 ** np.random.default_rng(4).uniform(-28.0, 6.0, 200000)
    got = np.zeros_like(x)
    f = A.lib().bysdf_audit_sqrt
    f.argtypes = [C.c_int64, C.c_void_p, C.c_void_p]
    assert f(len(x), A._ptr(x), A._ptr(got)) == 0
    ref = np.sqrt(x)
    assert np.all(np.abs(got - ref) <= np.spacing(ref))
    x[0], x[1] = 0.0, -1.0
    assert f(2, A._ptr(x), A._ptr(got)) == 0
    assert np.isnan(got[:2]).all()
