"""The steps that the waves of a factor workgroup share through LDS
(chol_steps.hpp), compiled for the host with one thread a lane and a schedule in
which one of them runs late."""
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
    exe = str(tmp_path_factory.mktemp("chol") / "chol_host_check")
    cmd = ["g++", "-O1", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "paper_2601_16379_amd", "csrc"),
           os.path.join(HERE, "chol_host_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return exe


def _run(exe, *args):
    r = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (args, r.stderr[-500:])
    return r.stdout.strip()


@pytest.mark.parametrize("n", [1, 5, 64])
@pytest.mark.parametrize("late", [-1, 3])
def test_diagonal_block_factor(driver, n, late):
    """L L^H within 8 n u of the block's largest diagonal."""
    word, err = _run(driver, "diag", n, -1, late).split()
    assert word == "factor" and float(err) <= 8 * n * 2.0 ** -53


@pytest.mark.parametrize("col", [0, 1, 4, 18, 63])
@pytest.mark.parametrize("late", [0, 1, 2, 3])
def test_breakdown_leaves_together(driver, col, late):
    """A breakdown is seen by every wave at the same barrier, whichever of them
    reads the flag late."""
    assert _run(driver, "diag", 64, col, late) == "breakdown"


@pytest.mark.parametrize("conj", [0, 1])
@pytest.mark.parametrize("late", [-1, 0, 1, 2, 3])
@pytest.mark.parametrize("rb", [1, 8, 9, 64])
def test_substitution(driver, rb, conj, late):
    """Unknowns that another lane of the quad stored are read after its store,
    whichever lane is late.  Two orders of the same sums: 64 roundings of terms
    that the 0.1-sized triangle keeps within a few times the result."""
    assert float(_run(driver, "tri", rb, conj, late)) <= 64 * 8 * 2.0 ** -53
