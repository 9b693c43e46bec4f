"""GPU tests of batches whose integrals take different paths in one step: other
numbers of histogram copies side by side in one launch, and bin counts on the
two sides of what the parallel bin adjustment's LDS holds, against the oracle's
and the single-integral runs, with the tolerances of the batch tests."""
import numpy as np
import pytest

import oracle as O
from paper_2202_01753_amd import mcubes as M
from paper_2202_01753_amd import workloads as W

pytestmark = pytest.mark.gpu

# bins per axis that the parallel adjustment takes (four arrays of them in LDS)
WIDE = M.MC_DEVICE_STEPS_MAX_BINS


def _check(results, probs, rel):
    for r, p in zip(results, probs):
        o = O.integrate(p)
        print(p["integrand"], p["dim"], p["nbins"], p["precision"], r["iterations"], flush=True)
        assert r["iterations"] == o["iterations"] and bool(r["converged"]) == o["converged"]
        assert r["estimate"] == pytest.approx(o["estimate"], rel=rel)
        assert r["error"] == pytest.approx(o["error"], rel=100 * rel)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_copies_of_every_number_in_one_launch(precision):
    # histogram and grid of d * nb bins take from 0.2 to 29 KB, so a workgroup's share of the LDS
    # (39 KB at four per CU) holds 16, 16, 8, 4, 2 and 1 copies
    sizes = [(1, 13), (2, 100), (3, 150), (4, 200), (5, 250), (6, 300)]
    probs = [(W.corner_peak if k % 2 else W.gauss_product)(d, 50 + k, maxcalls=40_000 + 1000 * k, nbins=nb, itmax=4,
                                                           seed=60 + k, precision=precision)
             for k, (d, nb) in enumerate(sizes)]
    probs += [W.symmetric_corner(4, a=1.0, maxcalls=50_000, nbins=90, itmax=4, one_d=1, seed=70, precision=precision),
              W.gauss_product(3, 71, maxcalls=60_000, nbins=64, itmax=5, ita=2, seed=71, precision=precision)]
    results, _ = M.batch_integrate(probs)
    _check(results, probs, 1e-10 if precision == "fp64" else 1e-5)


@pytest.mark.parametrize("nb", [WIDE - 1, WIDE, WIDE + 1, WIDE + 500])
def test_bin_adjustment_on_both_sides_of_its_lds(nb):
    # the integral with few bins shares the step's adjustment launch with the one with many
    probs = [W.corner_peak(1, 3, maxcalls=200_000, nbins=nb, itmax=4, seed=2),
             W.gauss_product(2, 4, maxcalls=50_000, nbins=50, itmax=4, seed=3)]
    results, _ = M.batch_integrate(probs)
    _check(results, probs, 1e-10)
    for r, p in zip(results, probs):
        one = M.integrate(p)
        assert r["estimate"] == pytest.approx(one.estimate, rel=1e-10)
        assert r["error"] == pytest.approx(one.error, rel=1e-8)
