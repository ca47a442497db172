"""The rounds of the one-launch iterations (csrc/coop.hip) as a model on the
CPU, over the library's own layout of slices and slots: built with g++ and
the sanitizers, see tests/sanitize/coop_rounds_driver.cpp."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "sanitize")
CSRC = os.path.join(ROOT, "paper_2602_23967_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ is needed")
def test_no_workgroup_waits_for_an_overwritten_round(tmp_path):
    exe = str(tmp_path / "rounds")
    subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                    os.path.join(CSRC, "prep.cpp"), os.path.join(HERE, "coop_rounds_driver.cpp"), "-o", exe], check=True)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and "rounds driver: 0 failure(s)" in p.stdout, (p.stdout + p.stderr)[-4000:]
