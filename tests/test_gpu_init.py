"""sky_init_box on trial states whose overlap is acceptable or not, on both
sides of 32 states, where its solver changes."""
import numpy as np
import pytest

from gpu_util import to_dev, to_host
from paper_1610_07522_amd import inputs, sky

pytestmark = pytest.mark.gpu

N = 8


def _box(m):
    return sky.Box(sky.desc_from_workload(inputs.small_workload("init", N, m, 1)))


def _trial(rng, m, lam):
    """States with overlap eigenvalues lam (volume element 1), and their
    Loewdin states."""
    q = np.linalg.qr(rng.standard_normal((1024, m)) + 1j * rng.standard_normal((1024, m)))[0].T
    z = np.linalg.qr(rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m)))[0]
    return ((z * np.sqrt(lam)) @ q).reshape(m, 2, N, N, N), z @ q


def _init(box, raw):
    one = np.zeros((1, 2, N, N, N), complex)
    one[0, 0, 0, 0, 0] = 1.0
    box.init_box(to_dev(raw), to_dev(one))


# the bound on an overlap eigenvalue is 1e-10 whatever the others are; squares of
# eigenvalues past 1e154 overflow
@pytest.mark.parametrize("m", [32, 33, 65])
@pytest.mark.parametrize("top,low,code", [
    (0.9e-10, 0.9e-10, sky.SKY_ERR_NOT_POSITIVE_DEFINITE), (1e-12, 1e-12, sky.SKY_ERR_NOT_POSITIVE_DEFINITE),
    (1e-5, 0.9e-10, sky.SKY_ERR_NOT_POSITIVE_DEFINITE), (1e160, 1e160, sky.SKY_ERR_NAN),
    (1.1e-10, 1.1e-10, 0), (1e-7, 1e-8, 0), (1e140, 1e138, 0)])
def test_scale_of_the_trial_states(m, top, low, code):
    rng = np.random.default_rng(900 + m)
    raw, want = _trial(rng, m, np.geomspace(top, low, m))
    box = _box(m)
    if code:
        with pytest.raises(sky.SkyError) as e:
            _init(box, raw)
        assert e.value.code == code
        return
    _init(box, raw)
    psi = to_host(box.view("psi")).reshape(m, -1)
    # rounding of the overlap (m ulps of its norm) over its smallest eigenvalue
    tol = 2.0 ** -52 * m * (top / low) + 1e-13
    assert np.abs(psi.conj() @ psi.T - np.eye(m)).max() <= tol
    assert np.abs(psi - want).max() <= tol
