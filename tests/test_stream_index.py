"""The reads of the one-token stream and the shares of its workgroups, on the CPU: both stand in headers of their own, and a host
program walks them over the shapes that the library takes.  (On the GPU a read behind a buffer shows only where the mapping ends.)"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("stream_index") / "driver")
    cmd = ["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2504_12285_amd", "csrc"), os.path.join(ROOT, "tests", "stream_index_driver.cpp"), "-o", exe]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout
    return exe


@pytest.mark.parametrize("what", ["activations", "issue", "cut"])
def test_stream_index(driver, what):
    run = subprocess.run([driver, what], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert run.returncode == 0 and "walk ok" in run.stdout, run.stdout
