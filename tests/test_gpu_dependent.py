"""Linearly dependent states are refused in both precisions, by every path that
orthonormalises: a state taken twice, a combination of the others, one of zeros,
one whose norm is below the bound of 1e-10; independent ones are taken."""
import numpy as np
import pytest
import torch

from paper_1610_07522_amd import inputs, sky

pytestmark = pytest.mark.gpu

N = 8
DTYPES = {sky.SKY_FP64: np.complex128, sky.SKY_MIXED: np.complex64}


def _states(m, kind, a, b):
    rng = np.random.default_rng(60 + m)
    x = rng.standard_normal((m, 2, N, N, N)) + 1j * rng.standard_normal((m, 2, N, N, N))
    x /= np.sqrt((abs(x) ** 2).sum(axis=(1, 2, 3, 4), keepdims=True))
    if kind == "twice":
        x[b] = x[a]
    elif kind == "combination":
        x[b] = np.delete(x, b, axis=0).sum(axis=0) / np.sqrt(m - 1)
    elif kind == "faint":
        x[b] *= 2.0 ** -40
    elif kind == "zero":
        x[b] = 0.0
    return x


def _orthonormalise(precision, x, how):
    dt = DTYPES[precision]
    phi = torch.from_numpy(x.astype(dt)).cuda()
    m = len(x)
    box = sky.Box(sky.desc_from_workload(inputs.small_workload("dependent", N, m, 1),
                                         precision=precision))
    out = torch.empty_like(phi)
    box.set_states(0, phi)
    if how == "loewdin":
        box.orthonormalize(0, phi, None, out)
    elif how == "ritz":
        spin = 1 + np.arange(2)[None, :, None, None, None]
        box.orthonormalize(0, phi, torch.from_numpy((spin * x).astype(dt)).cuda(), out)
    else:
        one = torch.zeros_like(phi[:1])
        one[0, 0, 1, 2, 3] = 1.0
        box.set_states(1, one)
        box.densities()
        getattr(box, how)(2)
        box.get_states(0, out)
    out = out.reshape(m, -1).to(torch.complex128).cpu().numpy()
    box.close()
    return out


# both sides of 32 states, where the solver changes, and of 128, where the pair
# lies in two tiles of the overlap
@pytest.mark.parametrize("m", [2, 5, 32, 33, 130])
@pytest.mark.parametrize("how", ["loewdin", "ritz", "iterate", "iterate_graph"])
@pytest.mark.parametrize("precision", sorted(DTYPES))
def test_dependent_states_are_refused(precision, how, m):
    cases = [("twice", 0, 1), ("twice", 0, m - 1), ("faint", 0, m - 1), ("zero", 0, m // 2)]
    if how in ("loewdin", "ritz"):   # the damped step is another one for each state
        cases.append(("combination", 0, m // 2))
    for kind, a, b in cases:
        with pytest.raises(sky.SkyError) as e:
            _orthonormalise(precision, _states(m, kind, a, b), how)
        assert e.value.code == sky.SKY_ERR_NOT_POSITIVE_DEFINITE, (kind, a, b)


@pytest.mark.parametrize("m", [2, 5, 32, 33, 130])
@pytest.mark.parametrize("how", ["loewdin", "ritz"])
@pytest.mark.parametrize("precision", sorted(DTYPES))
def test_independent_states_are_taken(precision, how, m):
    out = _orthonormalise(precision, _states(m, "independent", 0, 0), how)
    # rounding of the overlap (m ulps; mixed: 2^-20 for the split and the sums in
    # FP32) over its smallest eigenvalue, (1 - sqrt(m / 1024))^2 > 0.4
    tol = m * 2.0 ** -50 if precision == sky.SKY_FP64 else 2.0 ** -18
    assert np.abs(out.conj() @ out.T - np.eye(m)).max() <= tol
