"""A list's table cut into launches and blocks (csrc/smat_table.h), on the CPU: with launches small enough
that tables take many, every tile of every chunk and segment is taken once, in both block orders, and the
gradient norm's partials land in table order; at the real limit the pieces add up to the table."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2609_33437_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ is needed to build the test program")
def test_every_tile_once(tmp_path):
    exe = tmp_path / "table_check"
    build = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC,
                            os.path.join(HERE, "table_check.cpp"), "-o", str(exe)], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and run.stdout.strip() == "ok", run.stdout + run.stderr
