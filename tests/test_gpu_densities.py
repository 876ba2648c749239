"""Densities where the state chunks take several rounds of the card, against the
oracle: grids of which it holds few rows of workgroups at once."""
import numpy as np
import pytest

from gpu_util import rel_err, to_dev, to_host
from oracle import Grid
from oracle import physics as ph
from paper_1610_07522_amd import inputs, sky

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nn,np_,precision", [
    (48, 30, 5, sky.SKY_FP64), (48, 13, 13, sky.SKY_FP64), (64, 12, 4, sky.SKY_FP64), (64, 3, 1, sky.SKY_FP64),
    (48, 40, 10, sky.SKY_MIXED), (64, 12, 5, sky.SKY_MIXED)])
def test_densities(n, nn, np_, precision):
    mixed = precision == sky.SKY_MIXED
    w = inputs.small_workload("dens", n, nn, np_, init="rod", seed=60 + n, noise=0.1)
    raw = [p.astype(np.complex64 if mixed else np.complex128) for p in inputs.raw_states(w)]
    box = sky.Box(sky.desc_from_workload(w, precision=precision))
    for q in range(2):
        box.set_states(q, to_dev(raw[q]))
    box.densities()
    g = Grid(n, w.dx)
    # FP64: the parity bar of the step calls; mixed: FP32 derivatives, a few
    # hundred ulps of 2^-24 of the largest
    tol = 2e-5 if mixed else 1e-11
    for q in range(2):
        d = ph.densities(raw[q].astype(np.complex128), g)
        got = to_host(box.view("dens", q))
        for k, ref in enumerate((d.rho, d.tau)):
            assert rel_err(got[k], ref) <= tol, (q, k)
        assert rel_err(got[2:5], d.J) <= tol, q
