"""GPU test of the sampling kernels' FP64 exponential on its own: the integrand
values of a traced one-dimensional Gaussian pass (centre 0, width 1, so the
exponent is -x^2 rounded once) against extended precision.

The bound is the sum of the roundings in ulps of the result: 0.5 of the last
step, 0.18 of the sum before it, 0.20 of the reduced argument and 0.04 of the
rest reach 0.90 where they meet, plus 0.01 for the reference; a subnormal
result is rounded once more and has at least twice the spacing, 0.5 + 0.90 / 2."""
import numpy as np
import pytest

from paper_2202_01753_amd import mcubes as M
from paper_2202_01753_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("top", [1.0, 6.4, 26.6, 27.4])
def test_exponential_within_its_roundings(top):
    prob = W.gauss_product(1, 1, maxcalls=2_000_000, nbins=100, itmax=1, seed=77, lo=np.zeros(1), hi=np.array([top]))
    prob["params"] = np.array([0.0, 1.0])
    s = M.Sampler(prob)
    out = s.sample(0, M.init_grid(1, 100), trace_range=(0, s.m))["strace"]
    x, f = out[:, 2], out[:, 4]
    exact = np.exp(-(x * x).astype(np.longdouble))
    err = np.abs((f.astype(np.longdouble) - exact) / np.spacing(exact.astype(np.float64)).astype(np.longdouble))
    normal = exact >= np.finfo(np.float64).tiny
    print(top, "largest error", float(err[normal].max()), "ulp", flush=True)
    assert len(f) == 2_000_000 and float(err[normal].max()) <= 0.91
    if not normal.all():
        assert float(err[~normal].max()) <= 0.5 + 0.45 + 0.01


def test_exponential_at_the_ends_of_its_range():
    # far tails: every value 0 below the smallest subnormal, none negative or NaN
    prob = W.gauss_product(1, 1, maxcalls=20_000, nbins=100, itmax=1, seed=7, lo=np.zeros(1), hi=np.array([1e160]))
    prob["params"] = np.array([0.0, 1.0])
    s = M.Sampler(prob)
    out = s.sample(0, M.init_grid(1, 100), trace_range=(0, s.m))["strace"]
    assert (out[:, 4][out[:, 2] > 27.4] == 0.0).all()
