"""Dispatch orders, on the CPU, built with g++: the key preparation's workgroups (complete, and even over
the 8 XCDs: tests/host/prep_grid_test.cpp) and the row blocks of the sweeps (complete, and even over an
XCD's shader engines or the XCDs: tests/host/row_block_order_test.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("name,said", [("prep_grid_test", "prep grid ok"),
                                       ("row_block_order_test", "row block order ok")])
def test_every_workgroup_once_and_even(tmp_path, name, said):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is missing")
    exe = tmp_path / name
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra",
                        f"-I{ROOT}/paper_2608_27128_amd/csrc",
                        os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and said in r.stdout, r.stdout + r.stderr
