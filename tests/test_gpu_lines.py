"""Line and slice kernels of h psi and the damped step on every grid, in both
precisions, under a twist, against the oracle."""
import json

import numpy as np
import pytest

from gpu_util import rel_err, to_dev, to_host
from oracle import Grid
from oracle import physics as ph
from paper_1610_07522_amd import inputs, sky

pytestmark = pytest.mark.gpu

TWIST = (0.3, -0.7, 1.1)


@pytest.mark.parametrize("slices", [True, False])
@pytest.mark.parametrize("precision", [sky.SKY_FP64, sky.SKY_MIXED])
@pytest.mark.parametrize("n", [8, 16, 24, 32, 48, 64])
def test_h_and_damped_step(tmp_path, n, precision, slices):
    """h psi with <psi|h psi>, and the damped step with ||r||^2, by slices
    (where they fit) and by line passes."""
    torch = pytest.importorskip("torch")
    mixed = precision == sky.SKY_MIXED
    w = inputs.small_workload("lines", n, 3, 2, init="rod", seed=50 + n, noise=0.1)
    raw = [p.astype(np.complex64 if mixed else np.complex128) for p in inputs.raw_states(w)]
    box = sky.Box(sky.desc_from_workload(w, precision=precision, twists=[TWIST]))
    for q in range(2):
        box.set_states(q, to_dev(raw[q]))
    box.densities()
    form = "mixed" if mixed else "fp64"
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({f"h_lines/n{n}/{form}": -1 if slices else 32,
                                 f"damp_xy/n{n}/{form}": int(slices)}))
    box.autotune(str(cache))

    psi = [p.astype(np.complex128) for p in raw]
    g = Grid(n, w.dx).with_twist(TWIST)
    mf = ph.mean_field(*[ph.densities(p, g) for p in psi], g, w.params)
    # FP64: the parity bar of the step calls; mixed: FP32 transforms of a field
    # of order kmax^2 psi, a few hundred ulps of 2^-24
    tol = 2e-5 if mixed else 1e-11
    for q in range(2):
        m = raw[q].shape[0]
        dp, hp = to_dev(raw[q]), to_dev(np.zeros_like(raw[q]))
        phi, eps = to_dev(np.zeros_like(raw[q])), torch.zeros(m, dtype=torch.float64, device="cuda:0")
        r2 = torch.zeros_like(eps)
        box.apply_h(q, dp, hp, m, eps)
        ref = ph.apply_h(psi[q], mf[q], g)
        assert rel_err(to_host(hp), ref) <= tol, q
        dot = g.dV * np.einsum("asxyz,asxyz->a", psi[q].conj(), ref).real
        assert rel_err(to_host(eps), dot) <= tol, q
        # the step from the oracle's h psi, rounded to the form
        h = ref.astype(raw[q].dtype)
        box.damped_step(q, dp, to_dev(h), to_dev(dot), phi, m, r2)
        r = h.astype(np.complex128) - dot[:, None, None, None, None] * psi[q]
        mult = w.damp_x0 / (w.damp_e0 + mf[q].hb2m * g.k2_psi())
        step = np.fft.ifftn(mult * np.fft.fftn(r, axes=(2, 3, 4)), axes=(2, 3, 4))
        assert rel_err(to_host(phi), psi[q] - step) <= tol, q
        assert rel_err(to_host(r2), g.dV * (np.abs(r) ** 2).sum(axis=(1, 2, 3, 4))) <= tol, q
