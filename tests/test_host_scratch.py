"""What the C entry points do with their scratch where memory is short, under a
workspace cap and from call to call, with many devices and streams: api.cpp built with g++ against a small
fake of the HIP runtime (tests/host/scratch_check.cpp; no GPU code)."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2508_11467_amd", "csrc")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not installed")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    exe = str(tmp_path_factory.mktemp("host") / "scratch_check")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__", "-pthread",
           "-I", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    cmd += [os.path.join(CSRC, f) for f in ("api.cpp", "plan.cpp", "backtr_plan.cpp")]
    cmd += [os.path.join(HERE, "host", "scratch_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.mark.parametrize("case", ["out_of_memory", "kept", "few_reflectors", "captured", "many_devices",
                                  "reduction_under_a_cap", "streams", "captured_solve"])
def test_scratch(check, case):
    r = subprocess.run([check, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "0 failures" in r.stdout, (r.stdout + r.stderr)[-3000:]
