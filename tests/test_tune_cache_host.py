"""The autotuner's cache file (CPU only): entries written over another set of kernels do not count.
The harness is compiled with hipcc as host code."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2101_00941_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_entries_of_other_kernels_are_not_used(tmp_path):
    if not os.path.exists(HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "tune_cache_check")
    cmd = [HIPCC, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "host", "tune_cache_check.cpp"),
           os.path.join(CSRC, "plan.cpp"), os.path.join(CSRC, "tiling.cpp"), os.path.join(CSRC, "tune.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe, str(tmp_path / "tune.json")], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "ALL OK" in r.stdout, r.stdout + r.stderr
