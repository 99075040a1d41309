"""The planning of the multi-step block kernels (host code, built here with g++;
the checks are in block_plan_check.cpp)."""
import os
import shutil
import subprocess

import pytest

from block_geoms import EDGES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("block_plan") / "block_plan_check")
    subprocess.run([gxx, "-std=c++17", "-O2", "-D_GLIBCXX_ASSERTIONS",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_0911_0459_amd", "csrc"),
                    os.path.join(ROOT, "tests", "block_plan_check.cpp"), "-o", exe], check=True)
    return exe


def test_plans_from_kept_counts(exe):
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr


def test_lattices_at_the_tiles_edges_get_the_plans_they_name(exe):
    """So that a change of the planner cannot take the GPU tests off the edges: every
    shape, every number of steps per launch, and channels one row either side of what
    one, two and three tiles hold."""
    plans = set()
    for models, shape, K, column, g in EDGES:
        for m in models:
            got = subprocess.run([exe, m, *map(str, g)], capture_output=True, text=True, check=True).stdout.split()
            assert [int(v) for v in got][:2] == [shape, K], (m, g, got)
            assert column == 0 or int(got[2]) == column, (m, g, got)
            plans.add((m, shape, K))
            if column:
                halo, ry = 2 * K, 24 if shape == 2 or (shape == 1 and m == "b") else 32
                one = ry - halo - 1   # rows of a tile next to one wall
                assert g[4] in {1: [ry - 2], 2: [ry - 1, 2 * one], 3: [2 * one + 1]}[column]
    assert plans == ({("b", 0, K) for K in (2, 3, 4, 5)} | {("b", 1, K) for K in (2, 3)} |
                     {("b", 2, K) for K in (2, 3, 4, 5)} | {("v", 0, K) for K in (2, 3, 4, 5, 6)} |
                     {("v", 1, K) for K in (2, 3, 4)} | {("v", 2, K) for K in (2, 3, 4, 5)})
