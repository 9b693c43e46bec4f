"""CPU check of the batch engine's cut of a launch's work into shares that shrink:
every integral covered once and in order, no piece larger than the share it
lies in, no more pieces than the step area holds."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SHARES = [0.6, 0.3, 0.1]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("shares") / "check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-I", os.path.join(HERE, "..", "paper_2202_01753_amd", "csrc"),
                    os.path.join(HERE, "pins", "batch_shares_check.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("n,each,top", [(1, 1, 1), (1, 256, 10**9), (3, 1024, 5000), (192, 512, 10**6), (40, 7, 3)])
def test_shares_cover_every_integral(driver, n, each, top):
    rng = np.random.default_rng([n, each])
    m = rng.integers(1, top + 1, n)
    cost = rng.uniform(50.0, 4000.0, n)
    text = f"{n} {each} {len(SHARES)}\n{' '.join(map(str, SHARES))}\n" + "".join(
        f"{a} {c!r}\n" for a, c in zip(m.tolist(), cost.tolist()))
    lines = subprocess.run([driver], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    pieces = np.array([[int(x) for x in line.split()] for line in lines[:-1]])
    first = [int(x) for x in lines[-1].split()]
    assert len(pieces) <= n + each * len(SHARES)
    assert np.all(np.diff(pieces[:, 0]) >= 0)
    W, starts = float(m @ cost), np.concatenate([[0.0], np.cumsum(m * cost)])
    ends = np.cumsum(SHARES) * W
    for i in range(n):
        mine = pieces[pieces[:, 0] == i]
        assert pieces[first[i], 0] == i and (first[i] == 0 or pieces[first[i] - 1, 0] == i - 1)
        assert mine[0, 1] == 0 and mine[-1, 2] == m[i] and np.array_equal(mine[1:, 1], mine[:-1, 2])
        assert np.all(mine[:, 2] > mine[:, 1])
        for _, t0, t1 in mine:
            # the largest share that reaches past the piece's start (its cuts rounded to sub-cubes)
            level = min(int(np.searchsorted(ends, starts[i] + (t0 + 0.5) * cost[i])), len(SHARES) - 1)
            level = max(0, min(level, int(np.searchsorted(ends, starts[i] + (t0 - 1) * cost[i]))))
            assert (t1 - t0) * cost[i] <= W * SHARES[level] / each + 2 * cost[i] + 1e-9 * W
