"""How the model's formulas round, measured on the host: libbysdf_audit runs
the kernels' templates with chosen stages in single precision, so an
ill-conditioned form shows as an error far above its neighbours'."""
import ctypes as C

import numpy as np
import pytest

import precision_audit as A
from paper_2401_12724_amd import build as hip_build, workloads as W


@pytest.fixture(scope="module", autouse=True)
def audit_lib():
    if hip_build.stale():
        hip_build.build()


def _exit_error(eta):
    """rms relative error of E_yS with the exit refraction in single
    precision, around the direction that continues the incident one."""
    P = [W.default_params(eta=eta, B=0.0, beta=0.3)]
    q = W.queries(20000, 5, n_types=1, v_max=10.0)
    wi = np.asarray(q["wi"])
    d = -wi + 0.2 * np.random.default_rng(1).normal(size=wi.shape)
    q["wo"] = (d / np.linalg.norm(d, axis=0)).astype(np.float32)
    e = A.audit_eval(P, q, 0)[0][4].astype(np.float64)
    s = A.audit_eval(P, q, A.mask_of("exit"))[0][4].astype(np.float64)
    ok = e > 1e-3 * e.max()
    assert ok.sum() > 5000
    return np.sqrt(np.mean(((s - e)[ok] / e[ok]) ** 2))


def test_exit_refraction_conditioning():
    """The exit refraction's rounding changes smoothly with the index: over
    1.2 to 1.4 the half vector's length (at least eta - 1) doubles, so no
    error may exceed the one at 1.2 by more than sampling noise."""
    first = _exit_error(1.2)
    for eta in (1.249, 1.251, 1.3, 1.4):
        assert _exit_error(eta) <= 1.1 * first, eta


@pytest.mark.parametrize("eta", [1.1, 1.3, 1.55, 2.4])
def test_transmittance_rounding(eta):
    """The nodes' transmittance rounds no more than its textbook form, one
    quotient per polarisation (4 c e c_t / (c + e c_t)^2 and the like), does
    in single precision; 2 % covers the sampling of the rms over 10^6 cosines
    (0.1 %) and fused products."""
    n = 1 << 20
    c = np.random.default_rng(2).uniform(0.02, 1.0, n).astype(np.float32)
    got = np.zeros(n, np.float32)
    lib = A.lib()
    lib.bysdf_audit_transmittance.argtypes = [C.c_int64, C.c_void_p, C.c_float, C.c_void_p]
    assert lib.bysdf_audit_transmittance(n, A._ptr(c), eta, A._ptr(got)) == 0

    def form(c, e):
        one, two = c.dtype.type(1), c.dtype.type(2)
        ct = np.sqrt(one - (one - c * c) * (one / (e * e)))
        a, b = c + e * ct, e * c + ct
        return two * e * c * ct * (one / (a * a) + one / (b * b))

    exact = form(c.astype(np.float64), np.float64(np.float32(eta)))
    rms = lambda x: np.sqrt(np.mean(((x - exact) / exact) ** 2))
    assert rms(got) <= 1.02 * rms(form(c, np.float32(eta)))
