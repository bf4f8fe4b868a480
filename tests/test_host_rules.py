"""The rules that choose tile widths and kernels, checked on the CPU
(tests/native/rules_check.cpp)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1711_11296_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_rules(tmp_path):
    exe = str(tmp_path / "rules_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-DSHT_CHECK", "-I" + CSRC, "-I" + os.path.join(ROOT, "include"),
                        os.path.join(CSRC, "sht_plan.cpp"), os.path.join(CSRC, "sht_host.cpp"),
                        os.path.join(ROOT, "tests", "native", "rules_check.cpp"), "-pthread", "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and " 0 failures" in r.stdout, r.stdout
