"""GPU tests of the sampling launches that keep several copies of every
histogram bin side by side and spread a sub-cube's samples over several lanes:
one adjusting and one No-Adjust pass against the oracle's whole pass, with the
tolerances of the parity tests (summation order only, or an FP32
exponential's rounding)."""
import numpy as np
import pytest

import oracle as O
from paper_2202_01753_amd import mcubes as M
from paper_2202_01753_amd import workloads as W
from test_gpu_parity import _compare_totals, _positive_scale, _random_grid, _tol

pytestmark = pytest.mark.gpu


CASES = {
    # one sub-cube, whose samples go over the 64 lanes of one wave
    "d16 m1": lambda **k: W.corner_peak(16, 3, maxcalls=4001, nbins=7, **k),
    # 97 samples per sub-cube over 64 lanes: the last 31 lanes have one sample less
    "d10 p97": lambda **k: W.gauss_product(10, 4, maxcalls=100_000, nbins=50, **k),
    # 19 and 15 samples over 16 and 8 lanes, neither a multiple
    "d9 p19": lambda **k: W.corner_peak(9, 5, maxcalls=10_000, nbins=33, **k),
    "d8 p15": lambda **k: W.gauss_tables(8, 6, w_range=(0.1, 0.3), maxcalls=100_000, nbins=100, **k),
    # two samples over two lanes, a partial last wave
    "d2 p2": lambda **k: W.gauss_product(2, 7, maxcalls=9_800, nbins=100, **k),
    "d1 m2": lambda **k: W.gauss_product(1, 3, maxcalls=4, nbins=2, **k),
    # three samples, more sub-cubes than lanes: one lane each, 16 copies
    "d3 nb2": lambda **k: W.corner_peak(3, 8, maxcalls=1_000_000, nbins=2, **k),
    "d5 many": lambda **k: W.corner_peak(5, 9, maxcalls=2_500_007, nbins=101, **k),
    # bounds other than the unit cube, one row of contributions
    "d4 bounds one row": lambda **k: W.gauss_product(4, 10, maxcalls=60_001, nbins=64, one_d=True, lo=np.full(4, -1.0),
                                                    hi=np.array([1.0, 2.0, 0.5, 1.5]), **k),
    # the constant integrand: exact, without variance, however its samples are spread
    "d12 const": lambda **k: W.const(12, 1.5, maxcalls=40_000, nbins=16, **k),
}


@pytest.mark.parametrize("shape", [(0, 0), (64, 3), (768, 5)], ids=["default", "3x64", "5x768"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("case", CASES)
def test_pass_matches_oracle(case, precision, shape):
    prob = CASES[case](itmax=2, seed=31, precision=precision)
    threads, blocks = shape
    d, nb = prob["dim"], prob["nbins"]
    grid = _random_grid(d, nb, 17)
    if prob["one_d"]:
        grid = np.tile(grid[:nb + 1], d)
    s = M.Sampler(prob, blocks=blocks, threads=threads)
    print(case, precision, shape, M.launch_shape(s.bp), flush=True)
    for it, adjust in ((0, True), (1, False), (2, True)):
        gpu = s.sample(it, grid, adjust)
        gpu["nbins"] = nb
        ref = O.vsample(prob, it, grid, hist=adjust)
        _compare_totals(gpu, ref, _positive_scale(ref), f"{case} {precision} iter {it}", _tol(prob))
