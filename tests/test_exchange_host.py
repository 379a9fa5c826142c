"""Host model of the exchange between the workgroups of the tridiagonal
reduction (``csrc/exchange.h``): ``tests/exchange_check.cpp`` runs it with one
workgroup at a time held back, and no reader may find a word already written
for a later column than the one it waits for."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2005_06104_amd", "csrc")


def test_no_workgroup_is_overrun(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = tmp_path / "exchange_check"
    b = subprocess.run([cxx, "-O1", "-std=c++17", "-I" + CSRC, os.path.join(ROOT, "tests", "exchange_check.cpp"), "-o",
                        str(exe)], capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout[-2000:]
