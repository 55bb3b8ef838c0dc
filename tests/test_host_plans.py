"""The plans of the multi-step kernels and the rules of the default kernel
(csrc/host.cpp), built with AddressSanitizer and UndefinedBehaviorSanitizer
(g++, no GPU code) and swept over box sizes by tests/host_plan_driver.cpp."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2002_02503_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_plans_and_rules(tmp_path):
    exe = str(tmp_path / "host_plans")
    build = ["g++", "-std=c++20", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
             f"-I{CSRC}", os.path.join(ROOT, "tests", "host_plan_driver.cpp"), os.path.join(CSRC, "host.cpp"), "-o", exe]
    r = subprocess.run(build, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    assert "host plan driver: ok" in r.stdout
