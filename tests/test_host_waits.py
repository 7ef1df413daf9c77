"""The bounded waits of a grid's exchange (grid_sync.h) on the host: the header
is compiled with g++, the wavefront functions that it takes from block_util.h
replaced by those of a single thread."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2508_11467_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_waits_are_bounded(tmp_path):
    shutil.copy(os.path.join(CSRC, "grid_sync.h"), tmp_path)
    (tmp_path / "block_util.h").write_text("inline double wave_sum_last(double x) { return x; }\n")
    exe = str(tmp_path / "wait_check")
    cmd = ["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I", str(tmp_path),
           "-I", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"),
           os.path.join(HERE, "host", "wait_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "0 failures" in r.stdout, (r.stdout + r.stderr)[-3000:]
