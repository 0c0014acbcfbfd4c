"""The host layer's choices, on the CPU, built with g++ against the launcher stand-ins: the rule that
picks the sweep of a call over all columns (tests/host/sweep_rule_test.cpp) and the launches of a
short call (tests/host/launch_count_test.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_27128_amd", "csrc")
HOST = os.path.join(ROOT, "tests", "host")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.parametrize("name,said", [("sweep_rule_test", "sweep rule ok"),
                                       ("launch_count_test", "launch count ok")])
def test_host_choices(tmp_path, name, said):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime_api.h")):
        pytest.skip("g++ or the HIP headers are missing")
    exe = tmp_path / name
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{CSRC}",
                        f"-I{ROOT}/include", os.path.join(CSRC, "api.cpp"),
                        os.path.join(HOST, "stub_launchers.cpp"),
                        os.path.join(HOST, name + ".cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and said in r.stdout, r.stdout + r.stderr
