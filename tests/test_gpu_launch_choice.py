"""GPU tests of which kind of sampling launch a problem takes: the cases of the
tests named after a kind take that kind, with cases beside them where they
do not, and runs to a target take fused launches up to 200 bins only."""
import numpy as np
import pytest

import test_gpu_fused_runs as F
import test_gpu_launch_kinds as K
import test_gpu_staged as S
from launch_kinds import COPIES, FUSED, PLAIN, SPLIT, STAGED, STAGED_UNIT, launch_kind
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


STAGED_MORE = {
    "gauss d5 scaled fp64": (W.gauss_product, 5, 26, 2, 333, "fp64", False),
    "corner d10 scaled fp64": (W.corner_peak, 10, 5, 2, 300, "fp64", False),
    "tables d6 scaled fp64, two histogram copies": (W.gauss_tables, 6, 12, 2, 400, "fp64", False),
}
# (77 bins at d = 5 leave the LDS for copies of every bin: no staged launch)
STAGED_CASES = {k: v for k, v in S.CASES.items() if k != "gauss d5 scaled"}


@pytest.mark.parametrize("case", [*STAGED_CASES, *STAGED_MORE])
def test_cases_of_staged_passes_are_staged(case):
    make, d, g, p, nb, precision, unit = {**STAGED_CASES, **STAGED_MORE}[case]
    kw = dict(w_range=(0.1, 0.3)) if make is W.gauss_tables else {}
    if not unit:
        kw.update(lo=np.linspace(-0.25, 0.0, d), hi=np.linspace(1.0, 1.5, d))
    prob = make(d, 40 + d, maxcalls=p * g**d, nbins=nb, itmax=2, seed=19, precision=precision, **kw)
    assert _kind(prob) == (STAGED_UNIT if unit else STAGED) and _kind(prob, adjust=False) == PLAIN


@pytest.mark.parametrize("case", STAGED_MORE)
def test_more_staged_passes_match_the_oracle(case, monkeypatch):
    monkeypatch.setitem(S.CASES, case, STAGED_MORE[case])
    S.test_staged_pass_matches_oracle(case)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("case", K.CASES)
def test_cases_of_small_passes_are_split_or_have_copies(case, precision):
    prob = K.CASES[case](itmax=2, seed=31, precision=precision)
    want = COPIES if case in ("d3 nb2", "d5 many") else SPLIT
    assert _kind(prob) == want and _kind(prob, adjust=False) == want


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("case", F.CASES)
def test_cases_of_fused_runs_are_fused(case, precision):
    prob = _dev(F.CASES[case](seed=5, precision=precision))
    to_target = case in ("converges", "converges late", "target missed")  # (beyond 200 bins)
    assert _kind(prob, run=True) == (SPLIT if to_target else FUSED)


@pytest.mark.parametrize("blocks", [1, 7, 64])
@pytest.mark.parametrize("make,d,maxcalls,nb,precision", [
    (W.corner_peak, 9, 5_429_903, 58, "fp32"), (W.gauss_product, 16, 20_280_379, 21, "fp32"),
    (W.gauss_tables, 15, 183_386, 109, "fp64"), (W.gauss_product, 3, 132_288, 467, "fp64")])
def test_few_workgroups_asked_for_are_the_largest(make, d, maxcalls, nb, precision, blocks):
    # (one workgroup per CU at most: the most lanes are those of the largest workgroup)
    bp = M.BoundProblem(make(d, 3, maxcalls=maxcalls, nbins=nb, itmax=2, seed=5, precision=precision), blocks=blocks)
    for adjust in (True, False):
        assert M.launch_shape(bp, adjust)[:2] == (blocks, 1024)
