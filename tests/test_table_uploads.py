"""When tables are copied into a workspace (host only: the library's host code on a small runtime of the driver's own)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_06072_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("uploads") / "driver")
    srcs = [os.path.join(CSRC, f) for f in ("planner.cpp", "schedule.cpp", "trie.cpp", "api.cpp")]
    srcs.append(os.path.join(ROOT, "tests", "native", "uploads_driver.cpp"))
    build = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                            *srcs, "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    return exe


@pytest.mark.parametrize("check", ["captured", "graphs", "ahead"])
def test_table_uploads(driver, check):
    run = subprocess.run([driver, check], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, (run.stdout[-3000:], run.stderr[-3000:])
