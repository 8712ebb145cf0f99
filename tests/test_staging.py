"""The pinned staging that per-step tables are uploaded from (csrc/smat_staging.h), on the CPU against a
runtime that the test program plays: slot reuse waits for exactly that slot's upload, over several turns
of eight and of two slots; a wait neither waits for other work nor outlives a device that has failed."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2609_33437_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ is needed to build the test program")
def test_staging_protocol(tmp_path):
    exe = tmp_path / "staging_check"
    build = subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-pthread", "-I", CSRC,
                            os.path.join(HERE, "staging_check.cpp"), "-o", str(exe)], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and run.stdout.strip() == "ok", run.stdout + run.stderr
