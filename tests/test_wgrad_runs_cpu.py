"""The run arithmetic of the weight gradient's epilogue (csrc/runs.h) on the host, at the widest layers that the entries accept."""
import os
import subprocess

from conftest import ROOT
from paper_2302_05045_amd import _build


def test_runs_on_the_host(tmp_path):
    exe = str(tmp_path / "runs")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                           "-I", _build.CSRC, os.path.join(ROOT, "tests", "runs_driver.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and "0 failures" in out.stdout, (out.stdout + out.stderr)[-3000:]
