"""A solve that the device hands to the host reports its steps alike on both
sides of 32 states, where the solver changes."""
import numpy as np
import pytest

from gpu_util import to_dev
from paper_1610_07522_amd import inputs, sky

pytestmark = pytest.mark.gpu


# states too far from orthonormal for the series: no refinement step on the device
@pytest.mark.parametrize("m", [20, 32, 33, 40])
def test_steps_of_a_handed_over_solve(m):
    torch = pytest.importorskip("torch")
    w = inputs.small_workload("handover", 8, m, 0, init="rod", seed=5, noise=0.1)
    box = sky.Box(sky.desc_from_workload(w), stream=torch.cuda.Stream())
    rng = np.random.default_rng(m)
    q = np.linalg.qr(rng.standard_normal((1024, m)) + 1j * rng.standard_normal((1024, m)))[0].T
    psi = to_dev(1.5 * q.reshape(m, 2, 8, 8, 8) / w.dx ** 1.5)
    torch.cuda.synchronize()
    box.set_states(0, psi)
    box.densities()
    rep = box.iterate_graph(1, chunk=1)
    assert rep["eig_fallbacks"] == 1
    assert rep["eig_iters"] == 0
