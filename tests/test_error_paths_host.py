"""CPU check of the host driver's error paths on a stand-in for the HIP runtime:
whichever call fails, the entry points return MC_EDEVICE with nothing queued that
still reads the calling thread's page-locked memory or the caller's tables."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2202_01753_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    cxx, hip = shutil.which("g++"), "/opt/rocm/include"
    if cxx is None or not os.path.isdir(os.path.join(hip, "hip")):
        pytest.skip("no host C++ compiler or HIP headers")
    exe = str(tmp_path_factory.mktemp("errors") / "check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-w", "-pthread", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", "-I", hip,
                    "-I", os.path.join(HERE, "..", "include"), "-I", CSRC, os.path.join(CSRC, "mcubes_api.cpp"),
                    os.path.join(CSRC, "host.cpp"), os.path.join(HERE, "pins", "error_paths_check.cpp"), "-o", exe],
                   check=True)
    return exe


@pytest.mark.parametrize("tables", [0, 1])
@pytest.mark.parametrize("what", ["host", "device", "timed", "pass", "prepare"])
def test_errors_leave_nothing_queued(driver, what, tables):
    r = subprocess.run([driver, what, str(tables)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
