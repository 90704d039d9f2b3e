"""Host test of the heatmap kernels' logarithm table (built from the library's
own header; no GPU needed)."""

import os
import shutil
import subprocess

import pytest

from paper_2512_07009_amd import build as libbuild

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_ln_table(tmp_path):
    exe = str(tmp_path / "ln_table_test")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-I", libbuild.CSRC, os.path.join(HERE, "cpp", "ln_table_test.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "ln table ok" in r.stdout
