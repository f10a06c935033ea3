"""The column kernel's LDS indices, replayed on the host for every split that
the library plans (widths 3 to 16, single plates and batches, every step count
of a launch, every offset of a wall in its tile): the reflections at a wall stay
inside their velocity's plane and lattice column and off the lattice rows, and
every pull of an updated cell has a source."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_0904_4504_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_column_indices(tmp_path):
    lib = os.path.join(PKG, "liblbm.so")
    if not os.path.exists(lib):
        pytest.skip("library not built")
    exe = str(tmp_path / "column_plan_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-w",
                    "-I", os.path.join(PKG, "csrc"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROCM, "include"),
                    os.path.join(ROOT, "tests", "column_plan_check.cpp"), lib,
                    f"-Wl,-rpath,{PKG}", "-L", os.path.join(ROCM, "lib"), "-lamdhip64",
                    f"-Wl,-rpath,{os.path.join(ROCM, 'lib')}", "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[0]) > 10000
