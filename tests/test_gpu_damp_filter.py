"""The damping filter x0 / (E0 + T) is an FP64 quotient, rounded once to the
states' precision."""
import numpy as np
import pytest

from gpu_util import to_dev, to_host
from paper_1610_07522_amd import inputs, sky

pytestmark = pytest.mark.gpu


def _hard_quotients(rng, count):
    """(x0, E0) whose quotient lies a few FP64 ulps off the middle between two
    FP32 numbers, on either side."""
    e0 = rng.uniform(1.0, 200.0, count)
    mid = (2.0 * rng.integers(2 ** 23, 2 ** 24, count) + 1.0) * 2.0 ** -24   # 25 bits, odd
    x0 = mid * e0
    ulps = rng.choice([-24, -12, -6, -3, 3, 6, 12, 24], count)
    return x0 + ulps * np.spacing(x0), e0


def test_complex64_filter_is_the_rounded_fp64_quotient():
    """psi = 0 and a constant residual 1: only k = 0 is not zero, every transform
    of it is exact at 8^3, and phi is minus the filter's value there."""
    torch = pytest.importorskip("torch")
    n = 8
    one = to_dev(np.ones((1, 2, n, n, n), np.complex64))
    zero, phi = torch.zeros_like(one), torch.zeros_like(one)
    eps, r2 = (torch.zeros(1, dtype=torch.float64, device="cuda:0") for _ in range(2))
    w = inputs.small_workload("filter", n, 1, 1)
    for x0, e0 in zip(*_hard_quotients(np.random.default_rng(7), 128)):
        d = sky.desc_from_workload(w, precision=sky.SKY_MIXED)
        d.damp_x0, d.damp_e0 = x0, e0
        box = sky.Box(d)
        box.damped_step(0, zero, one, eps, phi, 1, r2)
        want = np.float32(x0 / n ** 3 / e0) * np.float32(n ** 3)
        got = to_host(phi)
        assert (got == -want).all(), (x0, e0, want, got[0, 0, 0, 0, 0])
