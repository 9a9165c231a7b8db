"""The order of a mixed step's workgroups: each of them once, prefill first (host only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_workgroup_once(tmp_path):
    exe = str(tmp_path / "mixed_order_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "paper_2602_06072_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "mixed_order_driver.cpp"), "-o", exe], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stdout
