"""GPU tests of one workspace that mc_prepare has filled once and runs with
other iteration counts (below and above the passes up to which steps go into the
sampling launches) or workgroups then use, in any order: every run against
a fresh one on a workspace of its own, with the tolerances of the device-steps tests."""
import ctypes as C

import pytest

from paper_2202_01753_amd import mcubes as M
from paper_2202_01753_amd import workloads as W
from test_gpu_device_steps import _dev, _same_run

pytestmark = pytest.mark.gpu

BASE = {
    "gauss d2": lambda **k: W.gauss_product(2, 21, maxcalls=10_000, nbins=100, **k),
    "corner d5 fp32": lambda **k: W.corner_peak(5, 22, maxcalls=60_000, nbins=60, precision="fp32", **k),
    "tables d4": lambda **k: W.gauss_tables(4, 23, w_range=(0.1, 0.3), maxcalls=50_000, nbins=40, **k),
}


def _bytes(bp, itmax, blocks=0):
    keep = bp.s.itmax, bp.s.ita, bp.s.blocks
    bp.s.itmax, bp.s.ita, bp.s.blocks = itmax, min(keep[1], itmax), blocks
    n = M.workspace_bytes(bp)
    bp.s.itmax, bp.s.ita, bp.s.blocks = keep
    return n


class _Filled(M.Workspace):
    """nbytes of device memory whose every double is a NaN and every word nonzero."""

    def __init__(self, nbytes):
        import torch
        self.nbytes = nbytes
        self.tensor = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")


def _check_runs(prob, runs, blocks_prepared=0):
    bp = M.BoundProblem(prob, blocks=blocks_prepared)
    ws = _Filled(max(_bytes(bp, itmax, blocks) for itmax, _, _, blocks in [(prob["itmax"], 0, 0, blocks_prepared)] + runs))
    M.prepare(prob, ws, bp=bp)
    for itmax, ita, tau, blocks in runs:
        print("itmax", itmax, "ita", ita, "tau", tau, "blocks", blocks, flush=True)
        bp.s.itmax, bp.s.ita, bp.s.tau_rel, bp.s.blocks = itmax, ita, tau, blocks
        p = dict(prob, itmax=itmax, ita=ita, tau_rel=tau)
        got = M.integrate(p, ws=ws, bp=bp, prepared=True)
        _same_run(got, M.integrate(dict(p, device_steps=False), blocks=blocks),
                  rel=1e-11 if prob["precision"] == "fp64" else 1e-9)


@pytest.mark.parametrize("device_steps", [False, True], ids=["host", "device"])
@pytest.mark.parametrize("name", BASE)
def test_iteration_counts_on_one_prepared_workspace(name, device_steps):
    prob = BASE[name](seed=31, itmax=10, ita=8, device_steps=device_steps)
    _check_runs(prob, [(10, 8, 0.0, 0), (100, 8, 0.0, 0), (10, 8, 0.0, 0), (65, 8, 0.0, 0), (64, 8, 0.0, 0),
                       (3, 3, 0.0, 0), (100, 0, 0.0, 0), (9, 9, 1e-9, 0)])


@pytest.mark.parametrize("device_steps", [False, True], ids=["host", "device"])
@pytest.mark.parametrize("name", BASE)
def test_prepared_with_many_iterations_run_with_few(name, device_steps):
    prob = BASE[name](seed=32, itmax=100, ita=8, device_steps=device_steps)
    _check_runs(prob, [(10, 8, 0.0, 0), (5, 5, 1e-9, 0), (100, 8, 0.0, 0), (2, 2, 0.0, 0)])


@pytest.mark.parametrize("device_steps", [False, True], ids=["host", "device"])
def test_workgroups_on_one_prepared_workspace(device_steps):
    prob = BASE["gauss d2"](seed=33, itmax=10, ita=8, device_steps=device_steps)
    runs = [(10, 8, 0.0, 0), (10, 8, 0.0, 3), (10, 8, 0.0, 0), (10, 8, 0.0, 40), (6, 6, 0.0, 0)]
    _check_runs(prob, runs)
    _check_runs(prob, runs, blocks_prepared=40)


@pytest.mark.parametrize("name", BASE)
def test_workspace_bytes_never_shrink_with_iterations(name):
    bp = M.BoundProblem(BASE[name](seed=34, itmax=1))
    sizes = [_bytes(bp, k) for k in (1, 2, 10, 63, 64, 65, 66, 100, 1000, 100_000)]
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("itmax", [5, 64, 65])
def test_run_on_exactly_the_bytes_asked_for(itmax):
    # device memory behind the workspace keeps its contents
    import torch
    prob = _dev(BASE["corner d5 fp32"](seed=35, itmax=itmax, ita=5))
    bp = M.BoundProblem(prob)
    n = M.workspace_bytes(bp)
    ws = _Filled(n + 65536)
    ws.nbytes = n
    got = M.integrate(prob, ws=ws, bp=bp)
    torch.cuda.synchronize()
    assert bool((ws.tensor[n:] == 0xFF).all())
    _same_run(got, M.integrate(dict(prob, device_steps=False)), rel=1e-9)
    res = M.Result(estimate=-3.0)
    code = M.lib().mc_integrate(bp.ref, ws.ptr, 1024, None, C.byref(res), None, None, None)
    assert code == M.EWORKSPACE and res.estimate == -3.0
