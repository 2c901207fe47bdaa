"""The arithmetic that sizes and cuts the interaction lists, compiled for the
host with g++ and its sanitizers (tests/list_math_driver.cpp)."""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_list_math_on_the_host(tmp_path):
    exe = tmp_path / "list_math"
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-Wall", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           f"-I{ROOT / 'paper_2107_07166_amd' / 'csrc'}", str(ROOT / "tests" / "list_math_driver.cpp"), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "list math ok" in r.stdout
