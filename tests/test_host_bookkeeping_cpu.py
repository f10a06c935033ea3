"""The host side's bookkeeping when calls fail, on a stand-in runtime of plain
host memory (tests/host_stub.cpp compiled with the library's host sources):
every step of every solve is launched once and in order, whatever failed
before."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_0904_4504_amd", "csrc")


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("stub") / "host_stub")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-w", "-pthread",
                    "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(rocm, "include"),
                    os.path.join(ROOT, "tests", "host_stub.cpp"),
                    *(os.path.join(CSRC, f) for f in ("api.cpp", "batch.cpp", "lattice.cpp",
                                                 "readout_pool.cpp")),
                    "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("check", ["refresh", "launch", "tile", "single", "beside", "pinned",
                                   "tables", "timing", "steps"])
def test_host(stub, check):
    r = subprocess.run([stub, check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
