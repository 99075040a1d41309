"""The planning of the multi-step block kernels (host code, built here with g++;
the checks are in block_plan_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plans(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "block_plan_check")
    subprocess.run([gxx, "-std=c++17", "-O2", "-D_GLIBCXX_ASSERTIONS",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_0911_0459_amd", "csrc"),
                    os.path.join(ROOT, "tests", "block_plan_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
