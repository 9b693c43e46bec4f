"""GPU tests of FP64 passes where the volume times nbins^dim, from which the
sampling kernels start a sample's Jacobian, is near or beyond the ends of the
range of doubles: one pass on a random grid against the oracle's, which
multiplies axis by axis (order of summation and rounding only), in the range
that starts from it and outside, where passes multiply axis by axis too."""
import numpy as np
import pytest

import oracle as O
from paper_2202_01753_amd import mcubes as M
from paper_2202_01753_amd import workloads as W
from test_gpu_parity import TOL, _random_grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("adjust", [True, False], ids=["adjust", "noadjust"])
@pytest.mark.parametrize("edge", [1e-100, 1e-69, 1e-66, 1.0, 1e60, 1e69])
def test_pass_over_a_tiny_or_vast_volume(edge, adjust):
    d, nb = 3, 40
    prob = W.gauss_product(d, 5, maxcalls=60_000, nbins=nb, itmax=2, seed=3,
                           lo=np.zeros(d), hi=np.full(d, edge))
    prob["params"] = np.asarray(prob["params"]) * edge
    grid = _random_grid(d, nb, 7)
    s = M.Sampler(prob)
    print(edge, M.launch_shape(s.bp), flush=True)
    gpu, ref = s.sample(0, grid, adjust), O.vsample(prob, 0, grid, hist=adjust)
    assert abs(gpu["I"] - ref["I"]) <= TOL * abs(ref["I"])
    if np.isfinite(ref["var"]):  # (squares of vast samples overflow, on both sides)
        assert abs(gpu["var"] - ref["var"]) <= TOL * abs(ref["var"])
    else:
        assert not np.isfinite(gpu["var"])
