"""Subspace matrices at the edges of their tiles, against numpy in FP64."""
import numpy as np
import pytest

from gpu_util import to_dev, to_host
from paper_1610_07522_amd import inputs, sky

pytestmark = pytest.mark.gpu


def _box(n, m, precision=sky.SKY_FP64):
    return sky.Box(sky.desc_from_workload(inputs.small_workload("edge", n, m, 1),
                                          precision=precision))


def _states(rng, m, n, dtype):
    x = rng.standard_normal((m, 2, n, n, n, 2))
    psi = (x[..., 0] + 1j * x[..., 1]).astype(np.complex128)
    psi /= np.sqrt((np.abs(psi) ** 2).sum(axis=(1, 2, 3, 4), keepdims=True))
    return psi.astype(dtype)


# 16: a block of the reduction; 64 and 128: tiles of the FP64 and plane products
@pytest.mark.parametrize("precision", [sky.SKY_FP64, sky.SKY_MIXED])
@pytest.mark.parametrize("m", [1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 129])
def test_overlap_and_h_matrices(m, precision):
    """I and H: entries, exact Hermitian symmetry, real diagonal."""
    n = 8
    mixed = precision == sky.SKY_MIXED
    rng = np.random.default_rng(100 + m)
    dt = np.complex64 if mixed else np.complex128
    phi, hphi = _states(rng, m, n, dt), _states(rng, m, n, dt)
    box = _box(n, m, precision)
    out = to_dev(np.zeros_like(phi))
    box.orthonormalize(0, to_dev(phi), to_dev(hphi), out)
    f, h = (x.reshape(m, -1).astype(np.complex128) for x in (phi, hphi))
    # unit vectors, 1024 products per entry: at most 1024 ulps of 1 in FP64;
    # the two-term split carries 2^-22 per operand of an entry at most 1
    tol = 1e-6 if mixed else 1024 * 2.0 ** -53
    for view, right in (("overlap", f), ("hsub", h)):
        got = to_host(box.view(view))
        ref = f.conj() @ right.T
        low = np.tril_indices(m)
        assert np.abs(got[low] - ref[low])[low[0] != low[1]].max(initial=0.0) <= tol
        # diagonals are summed in FP64 from the states in both forms
        assert np.abs(np.diag(got).real - np.diag(ref).real).max() <= 1024 * 2.0 ** -53
        assert np.array_equal(got, got.conj().T)


# 16: a Jacobi block; 32: one pair of blocks; 33, 49: an odd block count, padded
@pytest.mark.parametrize("m", [1, 2, 16, 17, 31, 32, 33, 48, 49, 97])
def test_jacobi_eigenpairs(m):
    """Loewdin of random states: the overlap's eigenpairs and psi = phi I^-1/2."""
    n = 8
    rng = np.random.default_rng(200 + m)
    phi = _states(rng, m, n, np.complex128)
    box = _box(n, m)
    out = to_dev(np.zeros_like(phi))
    box.orthonormalize(0, to_dev(phi), None, out)
    f = phi.reshape(m, -1)
    I = f.conj() @ f.T
    lam, z = np.linalg.eigh(I)
    # off-diagonal norm at most 1e-12 of the matrix norm (sqrt(m) to 2 sqrt(m))
    tol = 2e-12 * np.sqrt(m)
    assert np.abs(to_host(box.view("ritz")) - lam).max() <= tol
    v = to_host(box.view("evec"))
    assert np.abs(v.conj().T @ v - np.eye(m)).max() <= 1e-13 * max(m, 8)
    assert np.abs(I @ v - v * to_host(box.view("ritz"))).max() <= tol
    psi = to_host(out).reshape(m, -1)
    ref = ((z * lam ** -0.5) @ z.conj().T).T @ f
    assert np.abs(psi - ref).max() <= tol


# cluster sizes of a degenerate spectrum: none, pairs, shells, the widest cluster the
# refinement takes (48) and a wider one (Jacobi fallback)
@pytest.mark.parametrize("sizes", [[1] * 5, [2] * 8, [2, 12, 24], [1, 48, 3], [50, 2], [1] * 130,
                                   [2] * 40 + [24, 17, 24]])
def test_rayleigh_ritz_of_degenerate_levels(sizes):
    _check_degenerate(sizes)


# the one-workgroup solve (up to 32 states) at the edges of its two stored orders:
# clusters of one wave (to 16) and of the workgroup, odd ones, and none; 33 is past it
@pytest.mark.parametrize("sizes", [[1], [2], [3, 5, 7, 1], [16], [17], [1, 17, 13, 1], [16, 16], [31, 1],
                                   [3] * 10 + [2], [1] * 32, [2] * 16 + [1]])
def test_rayleigh_ritz_of_few_states(sizes):
    _check_degenerate(sizes)


# the last order on sub-tiles of one block and the first on two (ragged)
@pytest.mark.parametrize("m", [512, 513])
def test_rayleigh_ritz_of_many_states(m):
    _check_degenerate([1] * m)


def _check_degenerate(sizes):
    """Ritz values, U^H I U = 1 and U^H H U = diag for phi a small step off
    eigenstates of an operator with degenerate levels."""
    n, m = 8, sum(sizes)
    rng = np.random.default_rng(300 + m)
    q = np.linalg.qr(rng.standard_normal((1024, m)) + 1j * rng.standard_normal((1024, m)))[0].T
    lam = np.repeat(-60.0 + 3.0 * np.arange(len(sizes)), sizes)
    phi = q + 1e-4 * (rng.standard_normal(q.shape) + 1j * rng.standard_normal(q.shape))
    hphi = ((phi @ q.conj().T) * lam) @ q
    shape = (m, 2, n, n, n)
    box = _box(n, m)
    out, ritz = to_dev(np.zeros(shape, complex)), to_dev(np.zeros(m))
    box.orthonormalize(0, to_dev(phi.reshape(shape)), to_dev(hphi.reshape(shape)), out, ritz)
    I, H = phi.conj() @ phi.T, phi.conj() @ hphi.T
    low = np.linalg.inv(np.linalg.cholesky(I))
    ref = np.linalg.eigvalsh(low @ H @ low.conj().T)
    scale = np.abs(lam).max()
    assert np.abs(to_host(ritz) - ref).max() <= 1e-12 * scale * np.sqrt(m)
    u = to_host(box.view("umat"))
    assert np.abs(u.conj().T @ I @ u - np.eye(m)).max() <= 1e-12
    # the solvers stop at an off-diagonal Frobenius norm of 1e-12 of the norm
    d = u.conj().T @ H @ u
    assert np.linalg.norm(d - np.diag(np.diag(d))) <= 4e-12 * np.linalg.norm(lam)
    psi = to_host(out).reshape(m, -1)
    assert np.abs(psi - u.T @ phi).max() <= 1e-12


# 32: the last order left to the eigenvectors; condition numbers of the overlap that
# Newton's iteration takes (to 1e6) and one that it leaves to them
@pytest.mark.parametrize("cond", [1.0, 1e3, 1e6, 1e8])
@pytest.mark.parametrize("m", [1, 32, 33, 65, 150])
def test_initial_orthonormalisation(m, cond):
    """sky_init_box's Loewdin states against numpy, and their overlap."""
    n = 8
    rng = np.random.default_rng(500 + m)
    q = np.linalg.qr(rng.standard_normal((1024, m)) + 1j * rng.standard_normal((1024, m)))[0].T
    z = np.linalg.qr(rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m)))[0]
    phi = (z * np.logspace(0, -0.5 * np.log10(cond), m)) @ q
    raw = phi.reshape(m, 2, n, n, n)
    box = _box(n, m)
    box.init_box(to_dev(raw), to_dev(_states(rng, 1, n, np.complex128)))
    psi = to_host(box.view("psi")).reshape(m, -1)
    # rounding of I (m ulps of its norm) over its smallest eigenvalue
    tol = 2.0 ** -52 * m * cond + 1e-13
    assert np.abs(psi.conj() @ psi.T - np.eye(m)).max() <= tol
    assert np.abs(psi - z @ q).max() <= tol
