"""The dispatch order of the key preparation's workgroups, on the CPU: complete, and even over the
8 XCDs (tests/host/prep_grid_test.cpp, built with g++)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_workgroup_once_and_even_over_the_xcds(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is missing")
    exe = tmp_path / "prep_grid_test"
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra",
                        f"-I{ROOT}/paper_2608_27128_amd/csrc",
                        os.path.join(ROOT, "tests", "host", "prep_grid_test.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "prep grid ok" in r.stdout, r.stdout + r.stderr
