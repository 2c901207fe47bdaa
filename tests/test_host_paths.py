"""The library's host code when something is refused or fails, on the CPU: its host side
compiled with the address sanitizer and linked with a stand-in for the HIP
runtime that checks every launch (tests/fake_hip.cpp), driven by
tests/host_paths_driver.cpp."""
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
CSRC = ROOT / "paper_2107_07166_amd" / "csrc"
CLANG = Path("/opt/rocm/llvm/bin/clang++")
SCENARIOS = ["refused_memory", "wait_ran_out", "too_many_pairs", "too_many_rows", "first_walk_memory", "pass_sizes"]


def _run(cmd):
    r = subprocess.run([str(c) for c in cmd], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return r.stdout


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not CLANG.exists():
        pytest.skip("no ROCm compiler")
    tmp = tmp_path_factory.mktemp("host")
    # host code only: no device code is generated
    flags = ["-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O1", "-g", "-w",
             f"-I{ROOT / 'include'}", f"-I{CSRC}", f"-I{ROOT / 'tests'}", "-Xarch_host", "-fsanitize=address"]

    def compile_one(src):
        obj = tmp / (src.stem + ".o")
        _run([CLANG, *flags, "-c", src, "-o", obj])
        return obj

    srcs = sorted(CSRC.glob("*.hip")) + [ROOT / "tests" / "fake_hip.cpp", ROOT / "tests" / "host_paths_driver.cpp"]
    with ThreadPoolExecutor(4) as ex:
        objs = list(ex.map(compile_one, srcs))
    # the device code's symbols, which nothing reads
    names = sorted(set(re.findall(r"__hip_fatbin_\w+", _run(["nm", "-u", *objs]))))
    (tmp / "fatbin.c").write_text("".join(f"char {n}[64];\n" for n in names))
    _run(["gcc", "-c", tmp / "fatbin.c", "-o", tmp / "fatbin.o"])
    _run([CLANG, "-fsanitize=address", *objs, tmp / "fatbin.o", "-o", tmp / "driver"])
    return tmp / "driver"


@pytest.mark.parametrize("scenario", SCENARIOS)
def test_host_paths(driver, scenario):
    r = subprocess.run([str(driver), scenario], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert "host paths ok" in r.stdout
