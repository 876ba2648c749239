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


def _pair_box(mn, mp, stream=None):
    return sky.Box(sky.desc_from_workload(inputs.small_workload("init", N, mn, mp)), stream=stream)


def _pair(mn, mp, cond=100.0):
    rng = np.random.default_rng(950 + mn)
    return [_trial(rng, m, np.geomspace(2.0, 2.0 / cond, m))[0] for m in (mn, mp)]


def _overlap(raw):
    f = raw.reshape(raw.shape[0], -1)
    return f.conj() @ f.T


def _raw_eigenvalues(box, twin, q):
    """The eigenvalue buffer of a box without asking the box for it: the twin has
    the same workspace layout."""
    v = twin.view("ritz", q)
    off = v.data_ptr() - twin.ws.data_ptr()
    return box.ws[off:off + v.numel() * 8].view(v.dtype)


# the eigenvectors' side of the change of solver, its other side, and both in one box
@pytest.mark.parametrize("held", [False, True])
@pytest.mark.parametrize("mn,mp", [(32, 31), (33, 32), (32, 33), (65, 40)])
def test_overlap_eigenpairs_after_initialisation(mn, mp, held):
    raw = _pair(mn, mp)
    box = _pair_box(mn, mp)
    if held:   # buffers that the caller took before
        w, z = [box.view("ritz", q) for q in range(2)], box.view("evec", 1)
    box.init_box(*map(to_dev, raw))
    if not held:
        w, z = [box.view("ritz", q) for q in range(2)], box.view("evec", 1)
    for q in range(2):
        lam = np.linalg.eigvalsh(_overlap(raw[q]))
        # off-diagonal norm at most 1e-12 of the matrix norm
        tol = 2e-12 * np.linalg.norm(lam)
        assert np.abs(to_host(w[q]) - lam).max() <= tol, q
    I, v = _overlap(raw[1]), to_host(z)
    assert np.abs(v.conj().T @ v - np.eye(mp)).max() <= 1e-13 * mp
    assert np.abs(I @ v - v * to_host(w[1])).max() <= tol


def test_views_leave_the_states_alone():
    """The initial states do not depend on whether a caller has asked for eigenvalues."""
    raw = _pair(40, 35)
    out = []
    for held in (False, True):
        box = _pair_box(40, 35)
        if held:
            box.view("evec", 0)
        box.init_box(*map(to_dev, raw))
        out.append([to_host(box.view("psi", q)) for q in range(2)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)


def test_overlap_eigenvalues_give_way_to_the_next_solve():
    torch = pytest.importorskip("torch")
    mn, mp = 40, 35
    raw = _pair(mn, mp)
    lam = [np.linalg.eigvalsh(_overlap(r)) for r in raw]
    tol = [2e-12 * np.linalg.norm(v) for v in lam]
    asked, late, graph = _pair_box(mn, mp), _pair_box(mn, mp), _pair_box(mn, mp, torch.cuda.Stream())
    for b in (asked, late, graph):
        b.init_box(*map(to_dev, raw))
    asked.view("ritz", 0)
    asked.iterate(1)
    late.iterate(1)
    graph.iterate_graph(1)
    for q in range(2):
        ref = to_host(asked.view("ritz", q))
        assert np.abs(ref - lam[q]).max() > 1.0, q
        assert np.array_equal(to_host(late.view("ritz", q)), ref), q
        assert np.abs(to_host(graph.view("ritz", q)) - ref).max() <= 1e-9 * np.abs(ref).max(), q

    # a solve of one species into the caller's own buffer leaves both alone
    box = _pair_box(mn, mp)
    box.init_box(*map(to_dev, raw))
    phi = to_dev(raw[0])
    out, own = torch.empty_like(phi), torch.empty(mn, dtype=torch.float64, device="cuda:0")
    box.orthonormalize(0, phi, 3.0 * phi, out, own)
    assert np.abs(to_host(own) - 3.0).max() <= 1e-10
    v = to_host(box.view("evec", 0))
    assert np.abs(v.conj().T @ v - np.eye(mn)).max() <= 1e-13 * mn
    for q in range(2):
        assert np.abs(to_host(box.view("ritz", q)) - lam[q]).max() <= tol[q], q
    # and a second initialisation starts over
    again = _pair(mn, mp, 10.0)
    box.init_box(*map(to_dev, again))
    for q in range(2):
        ref = np.linalg.eigvalsh(_overlap(again[q]))
        assert np.abs(to_host(box.view("ritz", q)) - ref).max() <= tol[q], q


def test_eigenvalues_asked_for_during_a_capture():
    """They are left for the next request; the capture is not disturbed."""
    torch = pytest.importorskip("torch")
    raw = _pair(40, 35)
    dev = [to_dev(r) for r in raw]
    x = torch.zeros(64, device="cuda:0")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    box = _pair_box(40, 35, stream)
    box.init_box(*dev)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        x.add_(1.0)
        box.view("ritz", 0)
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert (x == k + 1.0).all()
    for q in range(2):
        lam = np.linalg.eigvalsh(_overlap(raw[q]))
        assert np.abs(to_host(box.view("ritz", q)) - lam).max() <= 2e-12 * np.linalg.norm(lam), q


# thirteen steps of at most 2.25 each: Newton's iteration takes 1e3 and cannot take 1e5;
# up to 32 states it is not tried
@pytest.mark.parametrize("cond,newton", [(1.0, True), (1e3, True), (1e5, False), (1e8, False)])
@pytest.mark.parametrize("m", [32, 33, 65, 150])
def test_solver_of_the_initialisation(m, cond, newton):
    """Which of the two solvers ran (only eigenvectors leave eigenvalues behind)."""
    raw = _trial(np.random.default_rng(980 + m), m, np.geomspace(1.0, 1.0 / cond, m))[0]
    box, twin = _box(m), _box(m)
    mark = _raw_eigenvalues(box, twin, 0)
    mark.fill_(-7.0)
    _init(box, raw)
    left = to_host(mark)
    if newton and m > 32:
        assert (left == -7.0).all()
    else:
        assert np.abs(left - np.linalg.eigvalsh(_overlap(raw))).max() <= 2e-12 * np.sqrt(m)


# where the iteration's last accepted start lies: each side must give Loewdin's states
@pytest.mark.parametrize("cond", [3e3, 1e4, 1.5e4, 2e4, 3e4])
@pytest.mark.parametrize("m", [33, 65, 150])
def test_edge_of_the_newton_iteration(m, cond):
    raw, want = _trial(np.random.default_rng(990 + m), m, np.geomspace(1.0, 1.0 / cond, m))
    box = _box(m)
    _init(box, raw)
    psi = to_host(box.view("psi")).reshape(m, -1)
    tol = 2.0 ** -52 * m * cond + 1e-13   # rounding of the overlap over its smallest eigenvalue
    assert np.abs(psi.conj() @ psi.T - np.eye(m)).max() <= tol
    assert np.abs(psi - want).max() <= tol
