"""The host's cutting of a row-lane launch, compiled for the CPU from the
library's own header (tests/cut/cut_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_random_batches_are_cut_soundly(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "cut_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-fsanitize=undefined,address",
                    "-fno-sanitize-recover", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROCM, "include"),
                    os.path.join(ROOT, "tests", "cut", "cut_check.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:verify_asan_link_order=0")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0, r.stdout + r.stderr[-3000:]
    assert r.stdout.startswith("ok ")
