"""Products of the fluxes where one side's sound speed plays no part
(tests/lagadj_cold.cpp, built with g++; no GPU) stay finite and agree with
central differences; the bound is that of the same check on ordinary states."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1408_3719_amd", "csrc")


@pytest.fixture(scope="module")
def deviations(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not available")
    exe = tmp_path_factory.mktemp("cold") / "lagadj_cold"
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run([gxx, "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "lagadj_cold.cpp"),
                    "-o", str(exe)], check=True, capture_output=True, timeout=300)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    return {name: float(dev) for name, dev in (ln.split() for ln in out.strip().splitlines())}


@pytest.mark.parametrize("name", ["rusanov_cold_left", "hll_cold_left", "hll_cold_left_upwind", "hll_upwind_in_time"])
def test_products_without_one_sides_sound_speed(deviations, name):
    assert deviations[name] < 1e-7
