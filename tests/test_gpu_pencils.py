"""h passes with twice the default pencils (384 or 512 threads): <psi|h psi> and
the FP64 diagonals of the mixed subspace matrices, summed over more than four
waves."""
import json

import numpy as np
import pytest

from gpu_util import rel_err, to_dev, to_host
from oracle import Grid
from oracle import physics as ph
from paper_1610_07522_amd import inputs, sky

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,lines,precision", [
    (16, 128, sky.SKY_FP64), (16, 128, sky.SKY_MIXED), (24, 64, sky.SKY_FP64), (24, 64, sky.SKY_MIXED),
    (32, 64, sky.SKY_FP64), (32, 64, sky.SKY_MIXED), (48, 64, sky.SKY_MIXED), (64, 64, sky.SKY_MIXED)])
def test_doubled_pencils(tmp_path, n, lines, precision):
    torch = pytest.importorskip("torch")
    mixed = precision == sky.SKY_MIXED
    w = inputs.small_workload("pencils", n, 5, 3, init="rod", seed=70 + n, noise=0.1)
    raw = [p.astype(np.complex64 if mixed else np.complex128) for p in inputs.raw_states(w)]
    box = sky.Box(sky.desc_from_workload(w, precision=precision))
    for q in range(2):
        box.set_states(q, to_dev(raw[q]))
    box.densities()
    form = "mixed" if mixed else "fp64"
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({f"h_lines/n{n}/{form}": lines, f"damp_xy/n{n}/{form}": 0}))
    assert box.autotune(str(cache))["h_lines"] == lines

    psi = [p.astype(np.complex128) for p in raw]
    g = Grid(n, w.dx)
    mf = ph.mean_field(*[ph.densities(p, g) for p in psi], g, w.params)
    tol = 2e-5 if mixed else 1e-11   # as the line passes' other pencil counts
    for q in range(2):
        m = raw[q].shape[0]
        hp = to_dev(np.zeros_like(raw[q]))
        eps = torch.zeros(m, dtype=torch.float64, device="cuda:0")
        box.apply_h(q, to_dev(raw[q]), hp, m, eps)
        got = to_host(hp).astype(np.complex128)
        assert rel_err(got, ph.apply_h(psi[q], mf[q], g)) <= tol, q
        # the sum itself, from the h psi that the kernel wrote: 2 n^3 FP64 products
        dot = g.dV * np.einsum("asxyz,asxyz->a", psi[q].conj(), got).real
        size = g.dV * np.einsum("asxyz,asxyz->a", np.abs(psi[q]), np.abs(got))
        assert (np.abs(to_host(eps) - dot) <= 4 * n ** 3 * 2.0 ** -53 * size).all(), q

    box.iterate(1)
    q = 1   # the subspace matrices hold the set last processed
    phi, hphi = (to_host(box.view(v, q)).astype(np.complex128) for v in ("phi", "hphi"))
    for view, right in (("overlap", phi), ("hsub", hphi)):
        diag = np.diag(to_host(box.view(view, q))).real
        ref = g.dV * np.einsum("asxyz,asxyz->a", phi.conj(), right).real
        size = g.dV * np.einsum("asxyz,asxyz->a", np.abs(phi), np.abs(right))
        assert (np.abs(diag - ref) <= 4 * n ** 3 * 2.0 ** -53 * size).all(), view
