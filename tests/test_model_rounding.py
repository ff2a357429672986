"""How the model's formulas round, measured on the host: libbysdf_audit runs
the kernels' templates with chosen stages in single precision, so an
ill-conditioned form shows as an error far above its neighbours'."""
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
