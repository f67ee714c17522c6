"""plan_wide's launch shapes are ones the wide kernel can run (CPU, sanitized)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_wide_plans_are_runnable(tmp_path):
    exe = str(tmp_path / "plan_wide_check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I",
                    os.path.join(ROOT, "paper_2505_18629_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "plan_wide_check.cpp"), "-o", exe], check=True,
                   capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
