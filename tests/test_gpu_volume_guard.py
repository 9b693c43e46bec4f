"""GPU tests of large FP64 passes just inside and just outside the range of
volumes whose Jacobian starts from the volume times nbins^dim: one pass on a
random grid against the oracle's, which multiplies axis by axis (order of
summation and rounding only), on the launch that each side is meant for."""
import numpy as np
import pytest

import oracle_pool as P
from launch_kinds import COPIES, PER_AXIS, PLAIN, STAGED, launch_kind
from paper_2202_01753_amd import mcubes as M
from paper_2202_01753_amd import workloads as W
from test_gpu_parity import TOL, _random_grid

pytestmark = pytest.mark.gpu

# dim, intervals per axis, bins, edge of the cube, kinds of an adjusting and of a No-Adjust pass.
# The volume times nbins^dim lies between 1e-200 and 1e200 for the first of each pair of edges,
# outside for the second.
CASES = [
    (3, 100, 40, 6e-69, COPIES, COPIES), (3, 100, 40, 5e-69, PER_AXIS, PER_AXIS),
    (3, 100, 40, 1.1e65, COPIES, COPIES), (3, 100, 40, 1.2e65, PER_AXIS, PER_AXIS),
    (3, 140, 40, 1.0, COPIES, PLAIN), (3, 140, 40, 1e-100, PER_AXIS, PER_AXIS),
    (5, 26, 333, 4e-43, STAGED, PLAIN), (5, 26, 333, 2e-43, PER_AXIS, PER_AXIS),
    (5, 26, 333, 2.5e37, STAGED, PLAIN), (5, 26, 333, 4e37, PER_AXIS, PER_AXIS),
]


@pytest.mark.parametrize("d,g,nb,edge,adjusting,no_adjust", CASES)
def test_pass_at_the_ends_of_the_volume_range(d, g, nb, edge, adjusting, no_adjust):
    prob = W.gauss_product(d, 5, maxcalls=2 * g**d, nbins=nb, itmax=2, seed=3, lo=np.zeros(d), hi=np.full(d, edge))
    prob["params"] = np.asarray(prob["params"]) * edge
    volume = np.prod(np.full(d, nb * edge, dtype=np.longdouble))
    assert (1e-200 < volume < 1e200) == (adjusting != PER_AXIS)
    s = M.Sampler(prob)
    assert s.g == g
    print(d, edge, launch_kind(s.bp), launch_kind(s.bp, adjust=False), M.launch_shape(s.bp), flush=True)
    assert (launch_kind(s.bp), launch_kind(s.bp, adjust=False)) == (adjusting, no_adjust)
    grid = _random_grid(d, nb, 7)
    for it, adjust in ((0, True), (1, False)):
        gpu, ref = s.sample(it, grid, adjust), P.vsample(prob, it, grid, hist=adjust)
        assert abs(gpu["I"] - ref["I"]) <= TOL * abs(ref["I"])
        if np.isfinite(ref["var"]):  # (squares of vast samples overflow, on both sides)
            assert abs(gpu["var"] - ref["var"]) <= TOL * abs(ref["var"])
        else:
            assert not np.isfinite(gpu["var"])
