"""GPU tests of device-steps runs whose steps lie inside the sampling launches
(small passes): whole runs against the host-steps run, with the tolerances of
the device-steps tests, and many runs of different lengths and ends on one
workspace, whose accumulators every run has to leave clear."""
import numpy as np
import pytest

from paper_2202_01753_amd import mcubes as M
from paper_2202_01753_amd import workloads as W
from test_gpu_device_steps import _dev, _same_run

pytestmark = pytest.mark.gpu

CASES = {
    "d1 two bins": lambda **k: W.gauss_product(1, 3, maxcalls=1000, nbins=2, itmax=4, **k),
    "d2 three bins": lambda **k: W.corner_peak(2, 4, maxcalls=9_800, nbins=3, itmax=5, **k),
    "d5 itmax 1": lambda **k: W.corner_peak(5, 5, maxcalls=30_000, nbins=40, itmax=1, **k),
    "d4 itmax 2": lambda **k: W.gauss_product(4, 6, maxcalls=30_000, nbins=65, itmax=2, **k),
    "d3 no-adjust tail": lambda **k: W.gauss_product(3, 7, maxcalls=50_000, nbins=64, itmax=6, ita=2,
                                                    lo=np.array([-1.0, 0.5, 2.0]), hi=np.array([1.0, 0.75, 9.0]), **k),
    "d3 no adjusting pass": lambda **k: W.corner_peak(3, 8, maxcalls=50_000, nbins=50, itmax=4, ita=0, **k),
    "d10 most bins": lambda **k: W.corner_peak(10, 9, maxcalls=100_000, nbins=160, itmax=4, **k),
    "d8 tables": lambda **k: W.gauss_tables(8, 10, w_range=(0.1, 0.3), maxcalls=100_000, nbins=100, itmax=4, **k),
    "m-Cubes1D": lambda **k: W.symmetric_corner(6, a=1.0, maxcalls=200_000, nbins=200, itmax=5, one_d=1, **k),
    "alpha": lambda **k: W.gauss_product(2, 11, maxcalls=20_000, nbins=100, itmax=6, alpha=0.7, **k),
    "64 passes": lambda **k: W.corner_peak(2, 12, maxcalls=5_000, nbins=32, itmax=64, **k),
    "converges": lambda **k: W.corner_peak(5, 14, maxcalls=200_000, nbins=100, itmax=12, tau_rel=1e-3, **k),
    "converges late": lambda **k: W.gauss_product(3, 15, maxcalls=50_000, nbins=100, itmax=30, tau_rel=1e-3, **k),
    "target missed": lambda **k: W.gauss_product(3, 15, maxcalls=50_000, nbins=100, itmax=5, tau_rel=1e-7, **k),
    "constant, exact": lambda **k: W.const(3, 2.5, maxcalls=8192, nbins=16, itmax=4, tau_rel=1e-3, **k),
}


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("case", CASES)
def test_fused_run_matches_host_steps(case, precision):
    prob = CASES[case](seed=5, precision=precision)
    print(case, precision, flush=True)
    # FP32: a boundary that moves by an ulp of FP64 can round to another float
    _same_run(M.integrate(_dev(prob)), M.integrate(prob), rel=1e-11 if precision == "fp64" else 1e-9)


def test_runs_of_every_end_on_one_workspace():
    base = _dev(W.corner_peak(4, 16, maxcalls=60_000, nbins=60, itmax=9, seed=9))
    bp = M.BoundProblem(base)
    ws = M.Workspace(bp)
    M.prepare(base, ws, bp=bp)
    for itmax, ita, tau in [(9, 9, 0.0), (9, 9, 2e-3), (1, 1, 0.0), (9, 3, 0.0), (2, 2, 0.0), (9, 9, 2e-3), (3, 0, 0.0),
                            (4, 4, 1e-9), (5, 5, 0.0), (9, 9, 0.0)]:
        bp.s.itmax, bp.s.ita, bp.s.tau_rel = itmax, ita, tau
        prob = dict(base, itmax=itmax, ita=ita, tau_rel=tau)
        got = M.integrate(prob, ws=ws, bp=bp, prepared=True)
        _same_run(got, M.integrate(dict(prob, device_steps=False)))


def test_non_finite_pass_ends_the_run_and_leaves_the_workspace_clean():
    d = 12
    prob = W.symmetric_corner(d, a=1.0, maxcalls=2**13, nbins=8, itmax=5, lo=np.zeros(d), hi=np.full(d, 1e4),
                              precision="fp32", device_steps=True)
    good = dict(prob, hi=np.ones(d))
    bp, bg = M.BoundProblem(prob), M.BoundProblem(good)
    ws = M.Workspace(bp)
    for tau in (0.0, 1e-9):
        bp.s.tau_rel = tau
        M.prepare(prob, ws, bp=bp)
        for _ in range(2):
            with pytest.raises(M.MCubesError) as e:
                M.integrate(prob, ws=ws, bp=bp, prepared=True)
            assert e.value.code == M.ENONFINITE
    got = M.integrate(good, ws=ws, bp=bg)
    _same_run(got, M.integrate(dict(good, device_steps=False)), rel=1e-9)
