"""The rule by which lr_lds takes a list for one whole list, on a CPU model of
its jumping rounds (tests/lds_list_driver.cpp, with the kernel's own word
functions): distances round a cycle grow past 16 bits and take any value, which
must never make a list without a tail look whole."""

import os
import subprocess

import pytest

from conftest import ROOT


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("lds") / "lds_list")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror",
                    "-I" + os.path.join(ROOT, "paper_1002_4482_amd", "csrc"),
                    os.path.join(ROOT, "tests", "lds_list_driver.cpp"), "-o", exe], check=True)

    def run(n, threads, shape, runs):
        r = subprocess.run([exe, str(n), str(threads), shape, str(runs)], check=True,
                           capture_output=True, text=True)
        return int(r.stdout)
    return run


# the workgroup of 1024 threads (one list, and batches up to 16384 nodes), and of
# 256 (batches up to 4096)
@pytest.mark.parametrize("n,threads", [(2, 1024), (65, 256), (1000, 256), (4000, 256),
                                       (4096, 256), (4096, 1024), (8000, 1024), (16383, 1024),
                                       (16384, 1024)])
def test_only_whole_lists_are_taken(model, n, threads):
    assert model(n, threads, "valid", 20) == 20
    assert model(n, threads, "back", 300) == 0
    assert model(n, threads, "circle", 50) == 0
    assert model(n, threads, "descending", 50) == 0
