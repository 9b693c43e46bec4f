"""GPU tests of which kind of sampling launch a problem takes."""
import pytest

from launch_kinds import COPIES, FUSED, SPLIT, launch_kind
from paper_2202_01753_amd import mcubes as M
from paper_2202_01753_amd import workloads as W
from test_gpu_device_steps import _dev, _same_run

pytestmark = pytest.mark.gpu


def _kind(prob, **kw):
    return launch_kind(M.BoundProblem(prob), **kw)


@pytest.mark.parametrize("d,nb,tau,fused", [(2, 100, 1e-3, True), (5, 40, 1e-3, True), (3, 67, 1e-3, False),
                                            (5, 60, 1e-3, False), (5, 60, 0.0, True), (10, 160, 0.0, True),
                                            (7, 229, 0.0, False)])
def test_runs_to_a_target_are_fused_up_to_200_bins(d, nb, tau, fused):
    # (in a run that ends after two passes the steps inside the launches cost more than they save)
    prob = _dev(W.corner_peak(d, 3, maxcalls=100_000, nbins=nb, itmax=6, tau_rel=tau, seed=4))
    assert _kind(prob, run=True) == (FUSED if fused else SPLIT)
    assert _kind(dict(prob, device_steps=False), run=True) == SPLIT
    _same_run(M.integrate(prob), M.integrate(dict(prob, device_steps=False)))


TARGET = {
    "two passes": lambda **k: W.corner_peak(4, 14, maxcalls=200_000, nbins=50, itmax=12, tau_rel=1e-2, **k),
    "converges": lambda **k: W.corner_peak(4, 14, maxcalls=20_000, nbins=50, itmax=12, tau_rel=5e-4, **k),
    "converges late": lambda **k: W.gauss_product(2, 15, maxcalls=5_000, nbins=100, itmax=40, tau_rel=5e-4, **k),
    "target missed": lambda **k: W.gauss_product(3, 15, maxcalls=50_000, nbins=66, itmax=5, tau_rel=1e-7, **k),
    "no-adjust tail": lambda **k: W.gauss_product(3, 7, maxcalls=50_000, nbins=64, itmax=20, ita=2, tau_rel=3e-4, **k),
}


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("case", TARGET)
def test_fused_run_to_a_target_matches_host_steps(case, precision):
    prob = TARGET[case](seed=5, precision=precision)
    assert _kind(_dev(prob), run=True) == FUSED
    got = M.integrate(_dev(prob))
    print(case, precision, got.iterations, got.converged, flush=True)
    _same_run(got, M.integrate(prob), rel=1e-11 if precision == "fp64" else 1e-9)
    assert got.converged == (case != "target missed") and (case != "two passes" or got.iterations == 2)
    assert 2 < got.iterations < prob["itmax"] or case in ("two passes", "target missed")
