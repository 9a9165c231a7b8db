"""The count by which the workgroups of a decode launch find the last of them: one arrival of each launch is the last, and the
count is back at zero when all have arrived, also after launches that overlapped.  Threads on the host in place of workgroups."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_count_returns_to_zero(tmp_path):
    exe = str(tmp_path / "arrival_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I" + os.path.join(ROOT, "paper_2602_06072_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "arrival_driver.cpp"), "-o", exe], check=True)
    for launches, parts in ((1, 4), (2, 2), (2, 3)):
        run = subprocess.run([exe, str(launches), str(parts)], capture_output=True, text=True, timeout=100)
        assert run.returncode == 0, run.stdout
