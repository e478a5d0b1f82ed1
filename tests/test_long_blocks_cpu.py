"""Pivot blocks of the long-row refactorization: builds
tests/long_blocks_driver.cpp with the host analysis and runs it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_blocks_stop_at_the_row_before_the_run(tmp_path):
    exe = tmp_path / "long_blocks"
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-mfma",
                    "-D_GLIBCXX_ASSERTIONS", os.path.join(ROOT, "tests", "long_blocks_driver.cpp"),
                    os.path.join(ROOT, "paper_2306_14337_amd", "csrc", "analyze.cpp"),
                    "-o", str(exe), "-pthread"], check=True, capture_output=True, text=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr
    ok, multi, with_link = res.stdout.split()
    assert ok == "ok" and int(multi) > 1000 and int(with_link) > 100
