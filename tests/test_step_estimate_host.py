"""How many global steps are queued between two status reads
(tests/step_estimate.cpp, built with g++; no GPU): as many as the instance
furthest behind needs by the steps taken so far, whichever instance that is."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1408_3719_amd", "csrc")


def test_steps_queued_in_named_situations(tmp_path):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not available")
    exe = tmp_path / "step_estimate"
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "step_estimate.cpp"), "-o", str(exe)],
                   check=True, capture_output=True, timeout=120)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    got = {name: int(n) for name, n in (ln.split() for ln in out.strip().splitlines())}
    assert got == {"no_step_yet": 1, "furthest_behind": 7, "limited": 8, "inside_one_step": 2,
                   "first_instance_done": 4, "next_target": 8, "first_instance_again": 4,
                   "bound_anew": 1, "nothing_to_do": 1}
