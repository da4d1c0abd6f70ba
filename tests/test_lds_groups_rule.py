"""How the two workgroups of a stretch of graphs share them, on a CPU model with
the kernel's own rules (tests/lds_groups_driver.cpp): one taker for every graph,
also where the pairs of a group pass 2^31 or the tables hold anything."""

import os
import subprocess

from conftest import ROOT


def test_every_graph_has_one_taker(tmp_path):
    exe = str(tmp_path / "lds_groups")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror",
                    "-I" + os.path.join(ROOT, "paper_1002_4482_amd", "csrc"),
                    os.path.join(ROOT, "tests", "lds_groups_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout
