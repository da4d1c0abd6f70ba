"""Sizes of the recorded walk, at sizes that no GPU test allocates and on random
batches (tests/record_plan_driver.cpp): strip numbers within 32 bits, memory
within its limit per node, and room for every strip of a group."""

import os
import subprocess

from conftest import ROOT


def test_sizes(tmp_path):
    exe = str(tmp_path / "record_plan")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror",
                    "-I" + os.path.join(ROOT, "paper_1002_4482_amd", "csrc"),
                    os.path.join(ROOT, "tests", "record_plan_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout
