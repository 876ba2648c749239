"""Phase timing changes no launch: the same bits with and without."""
import numpy as np
import pytest

from gpu_util import to_dev, to_host
from paper_1610_07522_amd import inputs, sky

pytestmark = pytest.mark.gpu

VIEWS = ("dens", "meanfield")


# more states than chunks of one species and of both; the most chunks (32), the card's
# own bound (24^3 FP64: 28, 32^3: 24 and 16), a species without states
@pytest.mark.parametrize("n,nn,np_,precision", [
    (8, 100, 37, sky.SKY_FP64), (16, 100, 40, sky.SKY_MIXED), (24, 70, 33, sky.SKY_FP64),
    (32, 70, 33, sky.SKY_FP64), (32, 70, 33, sky.SKY_MIXED), (48, 9, 5, sky.SKY_FP64),
    (48, 20, 7, sky.SKY_MIXED), (64, 9, 2, sky.SKY_MIXED), (16, 40, 0, sky.SKY_FP64)])
def test_timed_densities(n, nn, np_, precision):
    w = inputs.small_workload("timed", n, nn, np_, init="rod", seed=n, noise=0.05)
    raw = inputs.raw_states(w)
    out = []
    for timed in (False, True):
        box = sky.Box(sky.desc_from_workload(w, precision=precision))
        for q in range(2):
            if raw[q].shape[0]:
                box.set_states(q, to_dev(raw[q].astype(
                    np.complex64 if precision == sky.SKY_MIXED else np.complex128)))
        box.set_timing(timed)
        box.densities()
        out.append([to_host(box.view(v, q)) for v in VIEWS for q in range(2)] + [to_host(box.view("energy"))])
        if timed:
            t = box.timing()["densities"]   # the species' shares of the same launches
            assert t["ms_n"] > 0.0 and t["launches_n"] == t["launches_p"] == 1
            assert abs(t["ms_p"] * nn - t["ms_n"] * np_) <= 1e-6 * t["ms_n"] * nn
    assert np.abs(out[0][0]).max() > 0.0
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("precision", [sky.SKY_FP64, sky.SKY_MIXED])
def test_timed_iterations(precision):
    w = inputs.small_workload("timed", 16, 75, 40, init="rod", seed=3, noise=0.02)
    raw = inputs.raw_states(w)
    out = []
    for timed in (False, True):
        box = sky.Box(sky.desc_from_workload(w, precision=precision))
        box.init_box(*map(to_dev, raw))
        box.set_timing(timed)
        rep = box.iterate(2)
        out.append([np.array([rep["energy"], rep["residual"]])] +
                   [to_host(box.view(v, q)) for v in ("psi", "dens", "ritz") for q in range(2)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
