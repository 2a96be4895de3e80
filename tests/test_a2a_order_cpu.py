"""The XCD of every token's copies in the all-to-all dispatch (csrc/a2a_order.h) against the general placement
planner on the same workload (CPU only): random routings of 1-64 ranks, equal and mixed fan-outs."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_00867_amd", "csrc")
OUT = os.path.join(ROOT, "_build", "a2a_order")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_token_xcds_equal_the_planners():
    os.makedirs(OUT, exist_ok=True)
    exe = os.path.join(OUT, "a2a_order_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I" + CSRC,
                    "-I" + os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "c", "a2a_order_check.cpp"),
                    os.path.join(CSRC, "nap_planner.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    assert ", 0 mismatches" in r.stdout, r.stdout
