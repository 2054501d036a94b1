"""Host checks of the sweep's column plan and of the rules that hang on it, built with g++ under AddressSanitizer and
UndefinedBehaviorSanitizer (CPU only; see sanitize/column_driver.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_column_plan_under_sanitizers(tmp_path):
    exe = str(tmp_path / "column_driver")
    cmd = ["g++", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-g", "-O1",
           os.path.join(ROOT, "tests", "sanitize", "column_driver.cpp"),
           os.path.join(ROOT, "paper_1107_5719_amd", "csrc", "geometry.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and "column driver ok" in res.stdout, res.stdout + res.stderr
