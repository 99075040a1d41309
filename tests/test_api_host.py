"""Host logic of the library (lb_api.hip) without a GPU: its host half, built here,
on a HIP runtime of host memory that records launches, captures and allocations
(host_hip.h).  The checks are the functions of api_host_check.cpp."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCE = os.path.join(ROOT, "tests", "api_host_check.cpp")
CHECKS = re.findall(r'^\s*\{"(\w+)", \1\},$', open(SOURCE).read(), flags=re.M)


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(HIPCC):
        pytest.skip("no compiler")
    d = tmp_path_factory.mktemp("api_host")
    csrc = os.path.join(ROOT, "paper_0911_0459_amd", "csrc")
    inc = ["-I", os.path.join(ROOT, "include"), "-I", csrc, "-I", os.path.join(ROOT, "tests")]
    objects = []
    for src in (SOURCE, os.path.join(csrc, "lb_thermo.cpp"), os.path.join(csrc, "lb_analysis.cpp")):
        objects.append(str(d / (os.path.basename(src) + ".o")))
        subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-x", "hip", *inc,
                        "-c", src, "-o", objects[-1]], check=True)
    # (the device code that the objects refer to is not there)
    subprocess.run(["g++", *objects, "-no-pie", "-Wl,--unresolved-symbols=ignore-all", "-o", str(d / "check")], check=True)
    return str(d / "check")


@pytest.mark.parametrize("check", CHECKS)
def test_host_logic(exe, check):
    r = subprocess.run([exe, check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
