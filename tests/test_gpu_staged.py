"""GPU tests of staged adjusting passes (blocks of sub-cubes that share the digits
of their slow axes): one whole pass at the smallest lattices they are taken
for, against the oracle's pass over every sub-cube, on a random grid, with
the tolerances of the parity tests."""
import numpy as np
import pytest

import oracle_pool as P
from paper_2202_01753_amd import mcubes as M
from paper_2202_01753_amd import workloads as W
from test_gpu_parity import _compare_totals, _positive_scale, _random_grid, _tol

pytestmark = pytest.mark.gpu

# name: (make, dim, intervals per axis, samples per sub-cube, bins, precision, unit cube)
CASES = {
    "corner d5": (W.corner_peak, 5, 26, 2, 500, "fp64", True),
    "gauss d5 scaled": (W.gauss_product, 5, 26, 2, 77, "fp64", False),
    "tables d7 fp32, few bins": (W.gauss_tables, 7, 10, 2, 64, "fp32", True),
    "tables d6": (W.gauss_tables, 6, 12, 2, 500, "fp64", True),
    "tables d6 fp32 scaled": (W.gauss_tables, 6, 16, 2, 333, "fp32", False),
    "gauss d7": (W.gauss_product, 7, 10, 2, 401, "fp64", True),
    "corner d7 fp32": (W.corner_peak, 7, 11, 2, 500, "fp32", True),
    "gauss d9": (W.gauss_product, 9, 6, 2, 333, "fp64", True),
    "corner d9 fp32": (W.corner_peak, 9, 6, 2, 350, "fp32", True),
    "corner d10 three samples": (W.corner_peak, 10, 5, 3, 300, "fp64", True),
    "tables d10 fp32": (W.gauss_tables, 10, 5, 2, 310, "fp32", True),
}


@pytest.mark.parametrize("case", CASES)
def test_staged_pass_matches_oracle(case):
    make, d, g, p, nb, precision, unit = CASES[case]
    kw = dict(w_range=(0.1, 0.3)) if make is W.gauss_tables else {}
    if not unit:
        kw.update(lo=np.linspace(-0.25, 0.0, d), hi=np.linspace(1.0, 1.5, d))
    prob = make(d, 40 + d, maxcalls=p * g**d, nbins=nb, itmax=2, seed=19, precision=precision, **kw)
    grid = _random_grid(d, nb, 23)
    s = M.Sampler(prob)
    assert (s.g, s.p) == (g, p)
    print(case, M.launch_shape(s.bp), M.launch_shape(s.bp, adjust=False), flush=True)
    gpu = s.sample(1, grid, True)
    gpu["nbins"] = nb
    ref = P.vsample(prob, 1, grid, hist=True)
    _compare_totals(gpu, ref, _positive_scale(ref), case, _tol(prob))
    # a No-Adjust pass of the same workspace, then the adjusting one again
    s.sample(2, grid, False)
    again = s.sample(1, grid, True)
    assert again["I"] == gpu["I"] and again["var"] == gpu["var"]
    assert np.allclose(again["hist"], gpu["hist"], rtol=1e-12, atol=0)
