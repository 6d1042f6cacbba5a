"""The pool of idle workspaces (idle_pool.hpp), compiled for the host."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("pool") / "idle_pool_check")
    cmd = ["g++", "-O1", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "paper_2601_16379_amd", "csrc"),
           os.path.join(HERE, "idle_pool_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return exe


@pytest.mark.parametrize("what", ["sizes", "limits", "all", "nohost"])
def test_pool(driver, what):
    r = subprocess.run([driver, what], capture_output=True, text=True, timeout=60)
    assert (r.returncode, r.stdout.strip()) == (0, "ok")
