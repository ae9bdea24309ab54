"""The index arithmetic of the sums by distance bins, built with
UndefinedBehaviorSanitizer and checked on the CPU (tests/host/bin_checks.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_bin_arithmetic_under_sanitizer(tmp_path):
    exe = str(tmp_path / "bin_checks")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fsanitize=float-cast-overflow",
                    "-fno-sanitize-recover=all", os.path.join(HERE, "host", "bin_checks.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    assert "bin checks passed" in r.stdout
