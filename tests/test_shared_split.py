"""The split of shared segments in decode tables (host only: the schedule builder, compiled with g++)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_06072_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_items_cover_every_request_once(tmp_path):
    exe = str(tmp_path / "driver")
    srcs = [os.path.join(CSRC, f) for f in ("planner.cpp", "schedule.cpp", "trie.cpp", "api.cpp")]
    srcs.append(os.path.join(ROOT, "tests", "native", "shared_split_driver.cpp"))
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", *srcs, "-L/opt/rocm/lib", "-lamdhip64",
                    "-Wl,-rpath,/opt/rocm/lib", "-o", exe], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, (run.returncode, run.stdout)
