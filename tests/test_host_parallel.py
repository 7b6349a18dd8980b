"""The host loops of the plan (csrc/parallel.hpp) in sanitizer builds: an exception in
a worker thread (an allocation that fails in a large plan) reaches the caller, whose C
entry point reports it, instead of ending the process."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("sanitizer", ["address,undefined", "thread"])
def test_parallel_for(tmp_path, sanitizer):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = tmp_path / "parallel_test"
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", f"-fsanitize={sanitizer}",
           "-fno-sanitize-recover=all", "-pthread", "-I", os.path.join(ROOT, "paper_1311_4257_amd", "csrc"),
           os.path.join(ROOT, "tests", "host", "parallel_test.cpp"), "-o", str(exe)]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "parallel: ok" in r.stdout
