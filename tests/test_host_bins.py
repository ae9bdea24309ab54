"""The host side of the sums by distance bins, built with the sanitizers and
checked on the CPU: index arithmetic (tests/host/bin_checks.cpp), layouts and the
rules that choose the local sum's form (tests/host/form_checks.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2507_07823_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("name,sources", [("bin", []), ("form", ["wfp_forms.cpp", "wfp_host.cpp"])])
def test_bins_host_side_under_sanitizers(tmp_path, name, sources):
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fsanitize=float-cast-overflow",
                    "-fno-sanitize-recover=all", os.path.join(HERE, "host", f"{name}_checks.cpp"),
                    *[os.path.join(CSRC, s) for s in sources], "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    assert f"{name} checks passed" in r.stdout
