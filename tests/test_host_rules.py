"""Host-only checks of sizes and rules that decide how device work is laid out
and launched (`tests/host/*_check.cpp`), compiled with the host C++ compiler: no
GPU, no HIP runtime calls."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2606_24154_amd", "csrc")


@pytest.mark.parametrize("name", ["record_blocks", "eval_plan", "panel_rule"])
def test_rules(tmp_path, name):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / name)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC,
                    os.path.join(HERE, "host", name + "_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "checks passed" in r.stdout, r.stdout + r.stderr
