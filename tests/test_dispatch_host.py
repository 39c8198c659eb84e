"""CPU checks of the rules that choose a kernel or its launch shape, by a host
driver linked with the objects that build() made."""
import glob
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_0907_3022_amd", "csrc")
BUILD = os.path.join(ROOT, "paper_0907_3022_amd", "_build")
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    objs = sorted(glob.glob(os.path.join(BUILD, "*.o")))
    if not objs:
        pytest.fail("the library's objects are missing: run build() first")
    exe = str(tmp_path_factory.mktemp("dispatch") / "dispatch_check")
    obj = exe + ".o"
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                           "-I", CSRC, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-x", "hip", "-c",
                           os.path.join(ROOT, "tests", "sanitize", "dispatch_check.cpp"), "-o", obj])
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-o", exe, obj, *objs])
    return exe


@pytest.mark.parametrize("what", ["chain", "csr", "room", "walk", "holstein", "chunks", "shapes", "plan"])
def test_dispatch_rules(driver, what):
    r = subprocess.run([driver, what], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and ": 0 failures" in r.stdout, r.stdout
