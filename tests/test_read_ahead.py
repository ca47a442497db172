"""Results of a batch fetched in blocks (csrc/read_ahead.h) when host memory
runs out: no exception leaves the C entry point and the results are right;
built with g++ and the sanitizers, see tests/sanitize/read_ahead_driver.cpp."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_23967_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ is needed")
def test_no_exception_leaves_a_fetch(tmp_path):
    exe = str(tmp_path / "read_ahead")
    subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                    os.path.join(ROOT, "tests", "sanitize", "read_ahead_driver.cpp"), "-o", exe], check=True)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and "read-ahead driver: 0 failure(s)" in p.stdout, (p.stdout + p.stderr)[-4000:]
