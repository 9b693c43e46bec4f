"""The page-locked buffers that threads hold: a thread that ends leaves its
buffers to later ones.  On the CPU the pool with counted memory; on the GPU
runs from many short-lived threads, whose memory must not add up."""
import os
import shutil
import subprocess
import threading

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("pool") / "check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-pthread", "-I",
                    os.path.join(HERE, "..", "paper_2202_01753_amd", "csrc"),
                    os.path.join(HERE, "pins", "host_pool_check.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("what", ["one_after_another", "growing", "at_once", "without_memory"])
def test_pool(driver, what):
    r = subprocess.run([driver, what], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def _mapped_kb():
    """Memory of the GPU driver mapped into this process, page-locked host memory among it."""
    kb = 0
    with open("/proc/self/maps") as f:
        for line in f:
            if "/dev/dri/" in line or "/dev/kfd" in line:
                first, last = line.split()[0].split("-")
                kb += (int(last, 16) - int(first, 16)) // 1024
    return kb


@pytest.mark.gpu
def test_short_lived_threads_leave_nothing_behind():
    import torch

    from paper_2202_01753_amd import mcubes as M
    from paper_2202_01753_amd import workloads as W

    host = W.gauss_product(2, 3, maxcalls=10_000, nbins=50, itmax=3, seed=9)
    device = dict(host, device_steps=True)
    want = M.integrate(host).it_I.copy()
    results = []

    def work():
        # a fused run, one with launches of its own, and a host-steps run
        results.append((M.integrate(device), M.integrate(device, timing=True), M.integrate(host)))

    def threads(n):
        for _ in range(n):
            t = threading.Thread(target=work)
            t.start()
            t.join()
        torch.cuda.synchronize()

    threads(30)
    before = _mapped_kb()
    threads(300)
    grown = _mapped_kb() - before
    print("grown by", grown, "KB over 300 threads", flush=True)
    for rs in results:
        for r in rs:
            assert abs(r.it_I - want).max() <= 1e-11 * abs(want).max()
    # every thread's buffers of 64 KB would be 57 MB
    assert grown < 8192
